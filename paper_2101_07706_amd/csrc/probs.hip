// csgs_build_probs: importance weights over the neighbors of S_l (Section 4.1) and the skewed
// linear weighted sampling distribution (Section 4.2, Eq. 10) as an integer CDF.
//
// Kernels:
//   row_prefix     per tile of 1024 rows of S: degrees, their exclusive prefix (the flat edge
//                  numbering; tile offsets by the single-pass scan across blocks), CSR start of
//                  every row; the last tile leaves the row count and the edge counts for
//                  the kernels that follow
//   scan_edges     flat over the edges of S (chunks of 1024, a chunk's rows mapped to its positions in LDS, so
//                  hub rows and short rows cost the same per edge): square each edge value
//                  exactly, round to the fixed-point grid, add into a per-node 64-bit accumulator
//                  -- remote targets with fire-and-forget integer atomics; targets in the local id
//                  range (in calls with enough edges) are left grouped by tile for the next
//                  kernel, which sums them in LDS; flag the group of 8 node ids of the
//                  target (one 64-byte piece of the accumulator table) with a plain byte store, so
//                  that the candidate kernels fetch only touched pieces
//   cand_partials  sums of what the weight scan left for the local tiles; per tile of 1024 node ids: candidate count, local count, local and remote
//                  weight sums of the flagged words (unskewed, so they do not depend on s), and their
//                  sums per group of 64 tiles
//   scan_wide, bin_sums   the two for launches with many edges: all edges, remote ones too, are sorted by
//                  the block that sums their target and handed over; no scattered atomics
//   cand_emit      per tile: prefix = group sums before my group + tile sums before me in my
//                  group (plain loads: the producers are earlier kernels); the skew multiplier is
//                  fixed by the caller, or taken from the grand totals by the rule of Theorem 1
//                  (Eq. 12), or zero for remote nodes ("Local" version of Section 5.1); the
//                  tile's candidates are packed into LDS in id order (ballot popcount; of many tiles,
//                  four at a time, from the packed form that cand_partials leaves), then the
//                  packed list gets its skewed weights, their inclusive running sum and q, and goes
//                  out as contiguous runs of cand_id / cand_w / cdf / q; restores accumulator and
//                  flags to zero; the last tile writes the stats
#include <math.h>
#include "common.hpp"
#include "lookback.hpp"
#include "row_prefix.hpp"

namespace csgs {

// Rows given by the caller: one tile per block, grid = tiles of the row capacity; with a device-side
// count the blocks past it leave at once.
__global__ __launch_bounds__(256) void row_prefix(const int64_t *__restrict__ rowptr, int64_t n_nodes,
                                                  const int32_t *__restrict__ S, int32_t nS_bound,
                                                  const int32_t *__restrict__ nS_dev, const uint64_t *__restrict__ epoch,
                                                  uint64_t *__restrict__ ts_mem, int64_t ts_tiles,
                                                  int64_t *__restrict__ eoff, int64_t *__restrict__ rowstart,
                                                  int64_t *__restrict__ meta, int64_t edge_cap,
                                                  int2 *__restrict__ bound_note, int32_t *__restrict__ status, InstStride is)
{
    is = at_instance(is);
    bound_note = inst_ptr(bound_note, is.ws);
    S = inst_ptr(S, is.buf); nS_dev = inst_ptr(nS_dev, is.buf); status = inst_ptr(status, is.buf);
    epoch = inst_ptr(epoch, is.ws); ts_mem = inst_ptr(ts_mem, is.ws); eoff = inst_ptr(eoff, is.ws);
    rowstart = inst_ptr(rowstart, is.ws); meta = inst_ptr(meta, is.ws);
    const TileState<1> ts(ts_mem, ts_tiles, wait_limit(epoch));
    const int32_t nS = resolve_count(nS_bound, nS_dev);
    const int64_t n_tiles = row_tiles(nS);
    if ((int64_t)blockIdx.x >= n_tiles) return;
    row_prefix_tile(rowptr, n_nodes, S, nS, blockIdx.x, n_tiles, ts, call_tag(call_number(epoch), SLOT_ROWS), eoff, rowstart,
                    meta, edge_cap, bound_note, edge_cap / EDGE_TILE, status);
}

// Arguments of the hand-over from the weight scan to the candidate sums (see scan_edges).
struct Stage {
    uint64_t *e;        // [chunks * EDGE_TILE] weight * CAND_TILE + target id % CAND_TILE; a chunk's edges lie grouped by tile
    uint16_t *off;      // [chunks * SUB_STRIDE] per chunk and local tile: where its group begins (and the previous one ends)
    int64_t chunks;     // chunks the hand-over arrays can hold
    int32_t lo, hi;     // local id range
    int32_t tiles;      // tiles of CAND_TILE ids that meet it (0: every edge goes through device-scope atomics)
    int32_t max_split;  // blocks launched per tile
    int32_t adjacent;   // 1: a tile's blocks lie side by side (else one block of every tile after the other)
    int32_t n_inst;     // instances of the launch
    int32_t min_chunks; // chunks over all instances from which edges are handed over (0: whatever a chunk holds)
    int32_t below, bins; // wide form (scan_wide): bins before the local tiles, bins in all
    int32_t runs;       // most runs that are not whole ones (0: all are)
    unsigned long long *part;        // [tiles * max_split * CAND_TILE] sums of all but a tile's last block
    unsigned long long *part_flag;   // [tiles * max_split] tag of the call that left them
    uint64_t *gtot;     // [gtot_words] sums per group of tiles: the scan clears them for the candidate sums
    int64_t gtot_words;
};
// By the first wavefront of a scan: whether no instance's rows have more than 5 / 4 of the mean's edges.  `meta` and `epoch`: the first instance's.
__device__ inline void note_even_edges(int32_t n_inst, int64_t ws_stride, const int64_t *__restrict__ meta, uint64_t *__restrict__ epoch)
{
    static_assert(MAX_INSTANCES <= WAVE, "a lane per instance");
    const int lane = lane_id();
    const uint64_t mine = lane < n_inst ? (uint64_t)inst_ptr(meta, ws_stride * lane)[META_EDGES] : 0ull;
    const bool uneven = __any(mine * 4 * (uint64_t)n_inst > wave_sum(mine) * 5);
    if (lane == 0) epoch[EPOCH_EVEN] = uneven ? 0ull : 1ull;
}
// By the first block of a scan
__device__ inline void clear_group_sums(const Stage &stg, int64_t ws_stride)
{
    uint64_t *__restrict__ g = inst_ptr(stg.gtot, ws_stride);
    for (int64_t i = threadIdx.x; i < stg.gtot_words; i += blockDim.x) g[i] = 0ull;
}
// Local edges that a chunk must have to hand them over (more than EDGE_TILE: no chunk does).  Decided chunk by chunk from
// what there is, as the rows' degrees and the share of local targets may be anything, whatever the graph's mean and its
// partition.  What the hand-over saves grows with the local edges (their atomics, 23 G/s); what it costs is the sums' latency and
// a piece for every chunk: about 2.4 us and 6 ns a chunk, which an eighth of the edges does not bring in and half of them
// do from 160 chunks on.
__device__ inline uint32_t hand_over_from(const Stage &stg, int64_t n_chunks)
{
    if (stg.tiles <= 0) return EDGE_TILE + 1;
    if (stg.min_chunks == 0) return 0u;
    const int64_t all = n_chunks * stg.n_inst;   // every instance taken to have as many as the one at hand
    if (all < stg.min_chunks) return EDGE_TILE + 1;
    return EDGE_TILE / 7 + (all < 56 * EDGE_TILE ? 56u * EDGE_TILE / (uint32_t)all : 0u);
}
constexpr unsigned long long HAND_OVER_WEIGHTS = 1ull << 54;   // a weight that an entry can hold beside the 10 bits of the id (larger ones go through atomics)

// Fixed-point weight of an edge value: exact square (24 x 24 bit product) times a power of two, then round to nearest even;
// every candidate stays drawable.
__device__ inline unsigned long long edge_weight(float v, double scale)
{
    const double sq = (double)v * (double)v;
    const long long q = __double2ll_rn(sq * scale);
    return q < 1 ? 1ull : (unsigned long long)q;
}

// The weight scan, grid-stride over chunks of EDGE_TILE edges: map the chunk's positions to rows, fetch column and value of
// every edge, square, round.  An edge whose target lies outside the local id range is added to the per-node accumulator
// with a device-scope atomic.  The others -- most edges: the partition holds most neighbors -- are counting-sorted by the
// tile of their target inside the block and, where there are enough of them, written to the chunk's piece of the
// hand-over array: the next kernel has blocks per local tile, which add its groups up in LDS.  Scattered device-scope
// atomics run at about 23 G/s on this part whatever their scope or target range, and those of the remote edges are what
// bounds a large scan.  Integer sums: the result does not depend on which way an edge went or in what order.
// Nobody waits here, so there are as many blocks as the device holds (us, 512 blocks whose edges were summed by 2048-id
// owner blocks of the same launch / this: 6.7 M edges 211 / 83, 3.4 M 104 / 42, 1.0 M 50 / 17, eight mini-batches of
// 0.4 M 85 / 53; the sums then take 41, 26, 16 and 54 in cand_partials, which took 8 and, for the eight, 29).
__global__ __launch_bounds__(256) void scan_edges(const int32_t *__restrict__ colidx, const float *__restrict__ val,
                                                  int64_t n_nodes, int64_t nnz, int32_t shift_base,
                                                  const int64_t *__restrict__ meta, int64_t edge_cap,
                                                  const int64_t *__restrict__ eoff,
                                                  const int64_t *__restrict__ rowstart,
                                                  uint64_t *__restrict__ wtable, uint8_t *__restrict__ tileflag,
                                                  const int2 *__restrict__ bound_note,
                                                  uint64_t *__restrict__ epoch, int32_t *__restrict__ status, Stage stg, InstStride is)
{
    if (stg.n_inst > 1 && blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x < WAVE) note_even_edges(stg.n_inst, is.ws, meta, epoch);
    const InstBlock ib = inst_block_spread(is);
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block, n_blk = ib.blocks;
    constexpr int ITEMS = EDGE_TILE / 256;
    constexpr int BINS = SUB_MAX / WAVE;          // groups per lane of the counting sort
    static_assert(SUB_MAX % WAVE == 0 && EDGE_TILE <= 0xFFFF, "groups of a chunk");
    __shared__ EdgeMap<EDGE_TILE> map;
    __shared__ unsigned long long s_e[EDGE_TILE];
    __shared__ uint32_t hist[SUB_MAX + 1];
    meta = inst_ptr(meta, is.ws); eoff = inst_ptr(eoff, is.ws); rowstart = inst_ptr(rowstart, is.ws);
    wtable = inst_ptr(wtable, is.ws); tileflag = inst_ptr(tileflag, is.ws); bound_note = inst_ptr(bound_note, is.ws);
    stg.e = inst_ptr(stg.e, is.ws); stg.off = inst_ptr(stg.off, is.ws);
    status = inst_ptr(status, is.buf); epoch = inst_ptr(epoch, is.ws);
    ChunkRows rows = chunk_rows(bound_note, blk, (int64_t)blk + 1);   // (the grid stays within the notes; on its way beside the counts)
    const int32_t nS = (int32_t)meta[META_ROWS];
    const double scale = ldexp(1.0, shift_for_rows(shift_base, nS));
    const int64_t E = meta[META_EDGES];
    const int64_t n_chunks = (E + EDGE_TILE - 1) / EDGE_TILE;
    const uint32_t from = hand_over_from(stg, n_chunks);
    const int64_t n_staged = from <= EDGE_TILE ? stg.chunks : 0;   // (chunks beyond the arrays go through atomics)
    const unsigned long long call = call_number(epoch);
    const int32_t tile0 = stg.lo / CAND_TILE;
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);

    if (blk == 0) clear_group_sums(stg, is.ws);
    if (blk == 0 && threadIdx.x == 0 && meta[META_EDGES_TRUE] > edge_cap) atomicOr(status, CSGS_ST_EDGE_OVERFLOW);
    bool bad = false;
    for (int64_t t = blk; t < n_chunks; t += n_blk) {
        const int64_t c0 = t * EDGE_TILE;
        const int64_t c1 = (c0 + EDGE_TILE < E) ? c0 + EDGE_TILE : E;
        const bool staged = t < n_staged;
        if (staged)
            for (int i = threadIdx.x; i < SUB_MAX; i += blockDim.x) hist[i] = 0u;   // (its last readers are a barrier behind)
        const int32_t len = (int32_t)(c1 - c0);
        if (t != blk) rows = chunk_rows(bound_note, t, t + 1);
        (void)map_edges(map, eoff, rowstart, nS, c0, len, rows, first_rows(eoff, rowstart, nS, rows));   // (starts and ends with a barrier)
        const EdgeWords words = edge_words(map);
        // All of a thread's edges go through each step together -- their addresses, then their columns and
        // values with unconditional loads (an edge that does not exist reads entry 0 and is dropped) -- so
        // the loads of the four edges travel at the same time instead of one after the other.
        int64_t ek[ITEMS];
        bool live[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int32_t x = (int32_t)threadIdx.x + k * 256;
            ek[k] = 0;
            live[k] = x < len;
            const int64_t at = edge_address(map, words, __builtin_amdgcn_readfirstlane(wave + k * 4));
            if (live[k]) {
                ek[k] = at;
                if (ek[k] < 0 || ek[k] >= nnz) {   // only after a failed wait in the prefix kernel: stay inside the graph
                    bad = true;
                    ek[k] = 0;
                    live[k] = false;
                }
            }
        }
        int32_t ck[ITEMS];
        float vk[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            ck[k] = colidx[ek[k]];
            vk[k] = val[ek[k]];
        }
        unsigned long long qk[ITEMS];
        int32_t hb[ITEMS];    // tile of an edge that is handed over; -1: no edge, -2: device-scope atomic
        uint32_t hr[ITEMS];   // its place inside the group (any order)
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const bool sound = isfinite(vk[k]) && ck[k] >= 0 && ck[k] < n_nodes;
            if (live[k] && !sound) bad = true;
            hb[k] = -1;
            hr[k] = 0u;
            qk[k] = 0ull;
            if (!live[k] || !sound) continue;
            hb[k] = -2;
            qk[k] = edge_weight(vk[k], scale);
            if (staged && ck[k] >= stg.lo && ck[k] < stg.hi && qk[k] < HAND_OVER_WEIGHTS) {
                hb[k] = ck[k] / CAND_TILE - tile0;            // < stg.tiles <= SUB_MAX
                hr[k] = atomicAdd(&hist[hb[k]], 1u);
            }
        }
        if (staged) {
            __syncthreads();
            if (wave == 0) {   // counts -> begin of every group
                uint32_t cnt[BINS], sum = 0;
#pragma unroll
                for (int i = 0; i < BINS; ++i) {
                    cnt[i] = hist[lane * BINS + i];
                    sum += cnt[i];
                }
                const uint32_t incl = wave_inclusive_scan<uint32_t>(sum);
                const uint32_t n_local = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
                const bool take = n_local >= from;
                uint32_t ex = incl - sum;
#pragma unroll
                for (int i = 0; i < BINS; ++i) {
                    hist[lane * BINS + i] = ex;
                    if (lane * BINS + i <= stg.tiles) stg.off[t * SUB_STRIDE + lane * BINS + i] = (uint16_t)(take ? ex : 0u);
                    ex += cnt[i];
                }
                if (lane == WAVE - 1) {   // edges handed over by this chunk
                    hist[SUB_MAX] = take ? n_local : 0u;
                    if (stg.tiles == SUB_MAX) stg.off[t * SUB_STRIDE + SUB_MAX] = (uint16_t)(take ? n_local : 0u);
                    if (take && n_local) epoch[EPOCH_HANDED] = call;   // same value from every writer
                }
            }
            __syncthreads();
            const uint32_t n_handed = hist[SUB_MAX];
            if (n_handed) {
                // grouped in LDS first, then out in order: full 64-byte pieces instead of one scattered store per edge
#pragma unroll
                for (int k = 0; k < ITEMS; ++k)
                    if (hb[k] >= 0) s_e[hist[hb[k]] + hr[k]] = qk[k] * CAND_TILE + (unsigned)(ck[k] % CAND_TILE);   // < EDGE_TILE: the groups partition the chunk's local edges
                __syncthreads();
                for (uint32_t i = threadIdx.x; i < n_handed; i += blockDim.x) stg.e[t * EDGE_TILE + i] = s_e[i];
            } else {
#pragma unroll
                for (int k = 0; k < ITEMS; ++k)
                    if (hb[k] >= 0) hb[k] = -2;
            }
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (hb[k] != -2) continue;
            const int32_t c = ck[k];
            (void)__hip_atomic_fetch_add((unsigned long long *)&wtable[c], qk[k], __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
            tileflag[c >> 3] = 1;  // same value from every writer
        }
    }
    if (bad) atomicOr(status, CSGS_ST_BAD_EDGE_VALUE);
}

// The weight scan of a launch with many edges: every edge is handed over, so that none costs a scattered atomic.  A block sorts
// WIDE_EDGES edges at a time by the bin of their target -- the ids of one block of the candidate sums: a local tile, or four tiles
// elsewhere -- by a counting sort in LDS, and writes them out as one run.  The more edges at a time, the longer a bin's group in the run,
// which the sums read piece by piece.  What an entry does not hold (weights from WIDE_WEIGHTS on), crowded bins (below) and runs
// beyond the hand-over array go through the atomics.
constexpr int WIDE_CHUNKS = 16;                            // chunks of EDGE_TILE edges a run holds
constexpr int WIDE_EDGES = WIDE_CHUNKS * EDGE_TILE;
constexpr int WIDE_BLOCK = WIDE_EDGES / 16;                // 16 edges per thread
constexpr int WIDE_STEP = WIDE_BLOCK * 4;                  // mapped at a time
constexpr int WIDE_BINS = 4096;
constexpr int WIDE_STRIDE = WIDE_CHUNKS * SUB_STRIDE;      // entries per run of the groups' begins
constexpr int WIDE_IDS = CAND_TILE * 4;                    // most ids of a bin
constexpr int64_t BIN_FEW = 800;                            // expected edges per bin up to which a bin of several instances may be one wavefront's
constexpr int32_t BIN_ONE_WAVE = 490;                       // entries per bin outside the local range up to which it is
constexpr unsigned long long WIDE_WEIGHTS = 1ull << 52;
// A bin outside the local range is crowded, and its edges of a run go through the atomics, from this many edges over all runs, runs taken as alike: one
// block adds a bin up, at 0.4 ns an edge where runs are few and their groups long, at up to 1.4 where they are many.  Unless more of a run's bins are: then
// their blocks have enough company, and the atomics would cost as much.  (us of csgs_build_probs, narrow form / an eighth of a run as
// the line / this; 2.4 M nodes, a fifth of the edges remote.  204 runs: no bin crowded 88 / 72 / 65, one with 1 % of the edges 87 / 112 / 66, 5 % 86 / 307 / 70, 10 % 85 / 548 /
// 76, 12 % 86 / 640 / 79, ids by degree 370 / 119 / 89 (7 of it by the emission's two tiles a block).  436 runs: 153 / 106 / 101, 5 % 150 / 353 / 111, 12 % 144 / 714 / 128.  Eight
// instances of 24 runs: 126 / 90 / 90, 2 % 124 / 93 / 93, 5 % 122 / 111 / 108, 12 % 120 / 162 / 117.  Dearer for it than the narrow form, whose atomics
// travel beside its loads: all remote edges in a bin or eight, 204 runs 80 / 93 and 180 / 88, 436 runs 134 / 151 and 218 / 145.)
constexpr uint32_t WIDE_CROWD = 8192, WIDE_CROWD_FEW = 16384, WIDE_CROWD_RUN = 32;   // the latter: of a run at least
constexpr int WIDE_FEW_RUNS = WAVE, WIDE_CROWDED = 32;                             // most crowded bins of a run
constexpr int WIDE_STEP_CHUNKS = WIDE_STEP / EDGE_TILE;
// Steps of a run: four, with one instance no more than leave no more runs than there are compute units, each of which a run's block fills (us of
// csgs_build_probs with room for 65536 rows of 51 edges, whole runs / this: 1024 rows 42 / 34, 8192 57 / 48, 32768 65 / 59; with the emission's two tiles a block 32, 41, 52).
__device__ inline int run_steps_log2(int64_t n_chunks, const Stage &stg)
{
    const int64_t two = (int64_t)stg.runs * WIDE_STEP_CHUNKS * 2;   // chunks that runs of two steps hold
    return n_chunks > two ? 2 : (n_chunks > two / 2 ? 1 : 0);
}
__device__ inline int64_t run_count(int64_t n_chunks, const Stage &stg)
{
    const int steps = run_steps_log2(n_chunks, stg);
    return (n_chunks + (WIDE_STEP_CHUNKS << steps) - 1) / WIDE_STEP_CHUNKS >> steps;
}
static_assert(WIDE_CHUNKS == WIDE_STEP_CHUNKS * 4, "steps of a run");
static_assert(WIDE_STEP % EDGE_TILE == 0 && WIDE_BINS + 1 <= WIDE_STRIDE && WIDE_EDGES <= 0xFFFF && WIDE_STEP / WAVE <= WAVE, "runs of the wide form");

template <bool WHOLE>   // runs of WIDE_CHUNKS chunks, whatever there is
__global__ __launch_bounds__(WIDE_BLOCK) void scan_wide(const int32_t *__restrict__ colidx, const float *__restrict__ val, int64_t n_nodes,
                                                        int64_t nnz, int32_t shift_base, const int64_t *__restrict__ meta, int64_t edge_cap,
                                                        const int64_t *__restrict__ eoff, const int64_t *__restrict__ rowstart,
                                                        uint64_t *__restrict__ wtable, uint8_t *__restrict__ tileflag,
                                                        const int2 *__restrict__ bound_note, uint64_t *__restrict__ epoch,
                                                        int32_t *__restrict__ status, Stage stg, InstStride is)
{
    if (stg.n_inst > 1 && blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x < WAVE) note_even_edges(stg.n_inst, is.ws, meta, epoch);
    const InstBlock ib = inst_block_spread(is);
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block, n_blk = ib.blocks;
    constexpr int STEPS = WIDE_EDGES / WIDE_STEP, BINS = WIDE_BINS / WIDE_BLOCK;   // bins per thread
    __shared__ __attribute__((aligned(16))) union {   // (e is read two at a time)
        EdgeMap<WIDE_STEP> map;
        unsigned long long e[WIDE_EDGES];
    } u;
    __shared__ uint32_t hist[WIDE_BINS];
    __shared__ uint32_t s_scan[17];
    __shared__ int32_t n_crowded;
    meta = inst_ptr(meta, is.ws); eoff = inst_ptr(eoff, is.ws); rowstart = inst_ptr(rowstart, is.ws);
    wtable = inst_ptr(wtable, is.ws); tileflag = inst_ptr(tileflag, is.ws); bound_note = inst_ptr(bound_note, is.ws);
    stg.e = inst_ptr(stg.e, is.ws); stg.off = inst_ptr(stg.off, is.ws);
    status = inst_ptr(status, is.buf); epoch = inst_ptr(epoch, is.ws);
    const int32_t nS = (int32_t)meta[META_ROWS];
    const double scale = ldexp(1.0, shift_for_rows(shift_base, nS));
    const int64_t E = meta[META_EDGES];
    const int64_t n_chunks = (E + EDGE_TILE - 1) / EDGE_TILE;
    const int32_t steps = WHOLE ? STEPS : 1 << run_steps_log2(n_chunks, stg), per_run = steps * WIDE_STEP_CHUNKS;
    const int64_t n_runs = WHOLE ? (n_chunks + WIDE_CHUNKS - 1) / WIDE_CHUNKS : run_count(n_chunks, stg), n_staged = stg.chunks / WIDE_CHUNKS;
    uint32_t crowd = n_runs > WIDE_CROWD ? 0u : (n_runs > WIDE_FEW_RUNS ? WIDE_CROWD : WIDE_CROWD_FEW) / (uint32_t)(n_runs > 0 ? n_runs : 1);
    if (crowd < WIDE_CROWD_RUN) crowd = WIDE_CROWD_RUN;
    const unsigned long long call = call_number(epoch);
    const int32_t tile0 = stg.tiles ? stg.lo / CAND_TILE : 0x7FFFFFFF, tile1 = stg.tiles ? tile0 + stg.tiles : 0x7FFFFFFF;
    const int32_t past = stg.below + stg.tiles - tile1 / 4;   // of a tile past the local ones: its bin minus a quarter of it
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
    auto add = [&](int32_t c, unsigned long long q) {
        (void)__hip_atomic_fetch_add((unsigned long long *)&wtable[c], q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        tileflag[c >> 3] = 1;         // same values from every writer
        epoch[EPOCH_ADDED] = call;
    };
    if (blk == 0) clear_group_sums(stg, is.ws);
    if (blk == 0 && tid == 0 && meta[META_EDGES_TRUE] > edge_cap) atomicOr(status, CSGS_ST_EDGE_OVERFLOW);
    bool bad = false;
    for (int64_t run = blk; run < n_runs; run += n_blk) {
        const bool staged = run < n_staged;
        for (int i = tid; i < stg.bins; i += WIDE_BLOCK) hist[i] = 0u;   // (its last readers are a barrier behind)
        if (tid == 0) n_crowded = 0;
        // Which rows, and where they start, is asked for for all steps at once; columns and values of a step travel while the next one
        // is mapped.
        ChunkRows rows[STEPS];
        RowEdges mine[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int64_t t0 = run * per_run + s * WIDE_STEP_CHUNKS, t1 = t0 + WIDE_STEP_CHUNKS;
            rows[s] = s < steps && t0 < n_chunks ? chunk_rows(bound_note, t0, t1 < n_chunks ? t1 : n_chunks) : ChunkRows{0, 0};
        }
#pragma unroll
        for (int s = 0; s < STEPS; ++s) mine[s] = first_rows(eoff, rowstart, nS, rows[s]);
        int32_t col[STEPS][4];
        float v[STEPS][4];
        uint32_t live = 0;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (s >= steps) continue;
            const int64_t c0 = run * per_run * EDGE_TILE + (int64_t)s * WIDE_STEP, left = E - c0;
            const int32_t len = left <= 0 ? 0 : (left < WIDE_STEP ? (int32_t)left : WIDE_STEP);
            (void)map_edges(u.map, eoff, rowstart, nS, c0, len, rows[s], mine[s]);
            const EdgeWords words = edge_words(u.map);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int word = __builtin_amdgcn_readfirstlane(wave * 4 + k);
                const int64_t a = edge_address(u.map, words, word);
                const bool have = word * WAVE + lane < len, inside = a >= 0 && a < nnz;   // (outside only after a failed wait in the row pass)
                if (have && !inside) bad = true;
                live |= (uint32_t)(have && inside) << (s * 4 + k);
                const int64_t at = have && inside ? a : 0;
                col[s][k] = colidx[at];
                v[s][k] = val[at];
            }
        }
        unsigned long long entry[STEPS][4];
        uint32_t place[STEPS][4];   // bin << 16 | place inside its group (any order); all ones: nothing to hand over
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t c = col[s][k];
                const bool here = (live >> (s * 4 + k)) & 1u, sound = isfinite(v[s][k]) && c >= 0 && c < n_nodes;
                if (here && !sound) bad = true;
                place[s][k] = ~0u;
                entry[s][k] = 0ull;
                if (!here || !sound) continue;
                const unsigned long long q = edge_weight(v[s][k], scale);
                if (!staged || q >= WIDE_WEIGHTS) {
                    add(c, q);
                    continue;
                }
                const int32_t t = c / CAND_TILE;
                const int32_t b = t < tile0 ? t >> 2 : (t < tile1 ? stg.below + (t - tile0) : (t >> 2) + past);   // < stg.bins
                entry[s][k] = q * WIDE_IDS + (unsigned)(c % WIDE_IDS);
                place[s][k] = (uint32_t)b << 16 | atomicAdd(&hist[b], 1u);
            }
        }
        if (staged) {
            __syncthreads();
            // counts -> begin of every group; a crowded bin keeps an empty group and the top bit.  Both ways at once: with
            // the crowded bins' edges, and (upper half) without
            uint32_t cnt[BINS], sum = 0;
            bool heavy[BINS];
#pragma unroll
            for (int i = 0; i < BINS; ++i) {
                const int b = tid * BINS + i;
                cnt[i] = b < stg.bins ? hist[b] : 0u;
                heavy[i] = cnt[i] > crowd && (uint32_t)(b - stg.below) >= (uint32_t)stg.tiles;
                if (heavy[i]) atomicAdd(&n_crowded, 1);
                sum += cnt[i] | (heavy[i] ? 0u : cnt[i] << 16);
            }
            uint32_t n_handed;
            uint32_t ex = block_exclusive_scan<uint32_t>(sum, s_scan, &n_handed);
            const bool few_crowded = n_crowded <= WIDE_CROWDED;   // (complete since the scan's barriers)
            ex = few_crowded ? ex >> 16 : ex & 0xFFFFu;
            n_handed = few_crowded ? n_handed >> 16 : n_handed & 0xFFFFu;
#pragma unroll
            for (int i = 0; i < BINS; ++i) {
                const int b = tid * BINS + i;
                if (b < stg.bins) {
                    hist[b] = ex | (heavy[i] && few_crowded ? 0x80000000u : 0u);
                    stg.off[run * WIDE_STRIDE + b] = (uint16_t)ex;
                }
                ex += heavy[i] && few_crowded ? 0u : cnt[i];
            }
            if (tid == 0) {
                stg.off[run * WIDE_STRIDE + stg.bins] = (uint16_t)n_handed;
                if (n_handed) epoch[EPOCH_HANDED] = call;   // same value from every writer
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (place[s][k] == ~0u) continue;
                    const int32_t b = (int32_t)(place[s][k] >> 16);
                    const uint32_t begin = hist[b];
                    if (begin >> 31) {   // (not a local bin)
                        const int32_t first = (b < stg.below ? b : b - past) * WIDE_IDS;
                        add(first + (int32_t)(entry[s][k] % WIDE_IDS), entry[s][k] / WIDE_IDS);
                    } else {
                        u.e[begin + (place[s][k] & 0xFFFFu)] = entry[s][k];   // < WIDE_EDGES: the groups partition what is handed over
                    }
                }
            }
            __syncthreads();
            uint64_t *__restrict__ out = stg.e + run * WIDE_EDGES;
            for (uint32_t i = tid * 2u; i < n_handed; i += WIDE_BLOCK * 2u)
                *reinterpret_cast<ulonglong2 *>(&out[i]) = *reinterpret_cast<const ulonglong2 *>(&u.e[i]);   // (one past an odd end: inside the run)
        }
        __syncthreads();   // hist is cleared next
    }
    if (bad) atomicOr(status, CSGS_ST_BAD_EDGE_VALUE);
}

// Below this many chunks over all instances of a launch the atomics hide in the scan's latency (us for scan + candidate sums,
// atomics / hand-over, four edges in five local: 75 chunks 18 / 19, 426 chunks 36 / 24, 1004 chunks 56 / 33; one in two: 200
// chunks 20 / 21, 400 chunks 30 / 27; one in eight: 200 chunks 21 / 24, 800 chunks 50 / 53; one in 64: 800 chunks 50 / 68).
constexpr int32_t HAND_OVER_MIN_CHUNKS = 160;
// The wide form costs a sort of every edge and saves the scattered atomics and the sums' short reads (us of csgs_build_probs in the narrow / wide form; 2.4 M
// nodes, 150 local tiles: 1664 chunks 64 / 67, 2496 chunks 74 / 69, eight instances of 208 chunks 95 / 88, of 312 chunks 105 / 93, of 372 chunks 124 / 90, one of 6.6 K
// chunks 139 / 96; 200 K nodes: eight of 197 chunks 57 / 66, of 394 chunks 75 / 70).  Where the local range is too wide for the narrow form's hand-over, which then
// sends every edge through atomics, it pays much earlier (2 M nodes, 489 local tiles: 605 chunks 60 / 59, 1210 chunks 87 / 70, 3632 chunks 198 / 101).  With
// few bins their blocks leave compute units idle (30 K nodes, eight of 394 chunks: 73 / 82).  Beyond the hand-over array, whose other runs go through atomics, it is
// level on large graphs (2.4 M nodes, one edge in five remote: 9 M edges 196 / 160, 13 M 366 / 364, 20 M 668 / 630; 9.8 M nodes: 9 M 243 / 256, 11 M 329 / 311, 13 M
// 415 / 480, 20 M 727 / 732).
constexpr int64_t WIDE_MIN_CHUNKS = 2400, WIDE_MIN_CHUNKS_NARROW_OFF = 700;   // expected, over all instances
constexpr int64_t WIDE_RUNS = 256;                                            // of one instance: a run's block fills a compute unit
constexpr int64_t WIDE_MIN_BINS = 256;                                        // outside the local range, over all instances
// A tile's sums are split over several blocks while each block has this many edges left and the launch has SPLIT_BLOCKS
// of them at most, two per compute unit: a narrow local range has few tiles (29 tiles, 1 M edges: 31 us with a block
// per tile, 16 split by 7), and 150 tiles leave compute units idle (5.4 M edges: 49 / 40 us).  Shares below that only
// add the hop between the blocks (150 tiles, 0.35 M edges: 11 us with a block per tile, 14 split by 3).
constexpr int64_t SPLIT_MIN_EDGES = 4096;

// Skew policy, resolved on the device once the candidate counts are known.
struct SkewPolicy {
    int mode;          // 0: s_fx given; 1: Theorem 1 from (D, B), clamped to [16, s_fx_max]; 2: remote weight 0
    uint64_t s_fx;     // mode 0: local multiplier in 1/16 units
    double D;          // mode 1
    int64_t B;         // mode 1
    uint64_t s_fx_max; // mode 1
};

// Multipliers of local and remote weights (Eq. 10 numerators in 1/16 units).
__device__ inline void resolve_skew(const SkewPolicy &pol, uint64_t n_cand, uint64_t n_remote, uint64_t *m_local,
                                    uint64_t *m_remote)
{
    *m_remote = 16ull;
    if (pol.mode == 0) {
        *m_local = pol.s_fx;
    } else if (pol.mode == 1) {
        // s = D (|N(S_l)| - B) / |R| + 1/2 (Eq. 12), at least 1, no remote candidates -> 1
        double sk = 1.0;
        if (n_remote > 0) sk = pol.D * (double)((int64_t)n_cand - pol.B) / (double)n_remote + 0.5;
        if (!(sk >= 1.0)) sk = 1.0;
        double fx = floor(sk * 16.0 + 0.5);
        if (fx > (double)pol.s_fx_max) fx = (double)pol.s_fx_max;
        *m_local = (uint64_t)fx;
    } else {
        *m_local = 16ull;
        *m_remote = 0ull;
    }
}

constexpr int CAND_WORDS = CAND_TILE / WAVE;  // 16 words per tile, 4 per wave

// Tile sums and the sums of every group of 64 tiles.  Two kinds of blocks:
//  * a block of TILES tiles asks for the flags of all their words, then for their pieces of the table: two load latencies.
//  * where the weight scan may hand local edges over, every tile that meets the local range has blocks of its own.  If it
//    has done so, they first add up in LDS what the chunks left for the tile (64 chunks at a time per wavefront, one per
//    lane; each of the tile's blocks a share of the chunks, the last one all shares) and the last one stores the sums and
//    their touch flags: nobody else writes the local entries.  Bound by the latency of those reads; eight wavefronts per
//    block.
constexpr int CAND_PART_BLOCK = 512;
// Tiles per block of the first kind.  While all blocks with one tile each are on the device together, they are quickest
// (us per launch, four tiles / one: 4 tiles 6.6 / 5.2, 98 tiles 6.9 / 6.0, 256 tiles 7.5 / 5.6, 700 tiles 7.7 / 7.2); beyond
// that their number costs more than it gives (2392 tiles 10.6 / 14.1, eight times that 51 / 84; two tiles 11.8 and 62), and so
// it does with several instances (64 of 4 tiles 6.3 / 11).
constexpr int CAND_PART_TILES = 4;
constexpr int64_t CAND_PART_ONE = 1024;

// Sums of the edges that chunks [c_first, n_chunks) handed over for local tile `tile` into acc[CAND_TILE] (LDS, zeroed here).  A wavefront takes up to 64
// chunks at a time, one per lane, and walks through their groups as one sequence.  Called by all threads; ends with a barrier.
__device__ inline void sum_handed_over(unsigned long long *acc, const Stage &stg, int32_t tile, int64_t c_first, int64_t n_chunks)
{
    constexpr int U = 8;   // entries on their way per lane
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    for (int i = threadIdx.x; i < CAND_TILE; i += CAND_PART_BLOCK) acc[i] = 0ull;
    __syncthreads();
    const uint16_t *__restrict__ off = stg.off + tile;
    const uint64_t *__restrict__ e = stg.e;
    uint16_t beg, end;
    auto extents = [&](int64_t cb) {   // where my chunk's group lies in its piece
        const int64_t c = cb + lane;
        const uint16_t *p = off + (c < n_chunks ? c : 0) * SUB_STRIDE;   // (a share may hold no chunk at all)
        beg = p[0];
        end = p[1];
    };
    constexpr int WAVES = CAND_PART_BLOCK / WAVE;
    const int64_t want = (n_chunks - c_first + WAVES - 1) / WAVES;
    const int32_t per = want < WAVE ? (int32_t)want : WAVE;   // chunks per wavefront at a time
    int64_t cb = c_first + (int64_t)wave * per;
    extents(cb);
    for (; cb < n_chunks; cb += WAVES * per) {
        // entry j of the sequence belongs to the first lane whose running count exceeds j
        const int32_t n = (lane < per && cb + lane < n_chunks && beg <= end && end <= EDGE_TILE) ? (int32_t)end - (int32_t)beg : 0;
        const int32_t incl = wave_inclusive_scan<int32_t>(n);
        const int32_t first = (int32_t)beg - (incl - n) + lane * EDGE_TILE;   // it is entry first + j of the 64 chunks' pieces
        const int32_t total = __builtin_amdgcn_readlane(incl, WAVE - 1);
        const uint64_t *__restrict__ piece = e + cb * EDGE_TILE;
        extents(cb + WAVES * per);   // of the next chunks
        for (int32_t j0 = 0; j0 < total; j0 += U * WAVE) {
            uint64_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t j = j0 + u * WAVE + lane;
                int lo_l = 0, hi_l = WAVE - 1;
#pragma unroll
                for (int it = 0; it < 6; ++it) {
                    const int mid = (lo_l + hi_l) >> 1;
                    if (__shfl(incl, mid, WAVE) > j) hi_l = mid; else lo_l = mid + 1;
                }
                const int32_t pos = __shfl(first, lo_l, WAVE) + j;
                // unconditional (entry 0 stands in past the end and is dropped below), so that the steps' loads are on
                // their way together
                v[u] = piece[j < total ? pos : 0];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (j0 + u * WAVE + lane < total) atomicAdd(&acc[v[u] % CAND_TILE], (unsigned long long)(v[u] / CAND_TILE));
        }
    }
    __syncthreads();
}

// Lane i < 3 of a wavefront holds sum i of tile t in `mine`: left for cand_emit, and added to the sums of its group of 64 tiles, which the weight scan
// has cleared.  Nobody waits (with a last tile that waited for the others' flags and added them up: 59 against 55 us for an earlier bin_sums over eight instances,
// 1 % of the smallest step).
__device__ inline void publish_sum(int64_t t, int which, unsigned long long mine, unsigned long long *__restrict__ partial, uint64_t *__restrict__ gtot)
{
    partial[t * 4 + which] = mine;
    if (mine) (void)__hip_atomic_fetch_add((unsigned long long *)&gtot[t / LB_GROUP * 4 + which], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void publish_tile(int64_t t, unsigned long long mine, unsigned long long *__restrict__ partial, uint64_t *__restrict__ gtot)
{
    const int lane = lane_id();
    if (lane < 3) publish_sum(t, lane, mine, partial, gtot);
}

// PACK: the tiles are also put into the form that the packing kind of cand_emit reads, each tile's weights side by side at the start of its piece
// of the table and a bit per id in place of the groups' flags.
template <int TILES, bool PACK>
__global__ __launch_bounds__(CAND_PART_BLOCK, PACK ? 8 : 1) void cand_partials(uint64_t *__restrict__ wtable,
                                                     uint8_t *__restrict__ tileflag, int64_t n_words,
                                                     int64_t n_nodes, int64_t n_tiles, int32_t lo, int32_t hi,
                                                     const int64_t *__restrict__ meta, Stage stg,
                                                     int32_t blocks_below, const uint64_t *__restrict__ epoch,
                                                     unsigned long long *__restrict__ partial,
                                                     uint64_t *__restrict__ gtot, int32_t *__restrict__ status, InstStride is)
{
    const InstBlock ib = inst_block(is, epoch[EPOCH_EVEN] != 0);
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block;
    constexpr int WAVES = CAND_PART_BLOCK / WAVE, W = TILES * CAND_WORDS / WAVES;   // words per wavefront
    __shared__ uint64_t lds[WAVES][3];
    __shared__ unsigned long long acc[CAND_TILE];
    __shared__ __attribute__((aligned(8))) uint8_t s_bits[PACK ? WAVES : 1][W * 8];   // a wavefront's groups: a bit per id
    wtable = inst_ptr(wtable, is.ws); tileflag = inst_ptr(tileflag, is.ws); epoch = inst_ptr(epoch, is.ws);
    partial = inst_ptr(partial, is.ws); gtot = inst_ptr(gtot, is.ws);
    status = inst_ptr(status, is.buf); meta = inst_ptr(meta, is.ws);
    stg.e = inst_ptr(stg.e, is.ws); stg.off = inst_ptr(stg.off, is.ws);
    stg.part = inst_ptr(stg.part, is.ws); stg.part_flag = inst_ptr(stg.part_flag, is.ws);
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const unsigned long long tag = call_tag(call_number(epoch), SLOT_CAND);
    // blocks in the order of their tiles: blocks_below of TILES tiles, max_split per tile that meets the local range, TILES again
    const int64_t tile0 = stg.lo / CAND_TILE;
    int64_t t0, t1;
    const int32_t b = (int32_t)blk - blocks_below;
    const int32_t own_blocks = stg.tiles * stg.max_split;   // at most SPLIT_BLOCKS
    const bool own = b >= 0 && b < own_blocks;
    const uint32_t per_step = stg.adjacent ? (uint32_t)stg.max_split : (uint32_t)stg.tiles;
    const uint32_t step_own = own ? (uint32_t)b / per_step : 0u, rest_own = own ? (uint32_t)b % per_step : 0u;
    const uint32_t tile_own = stg.adjacent ? step_own : rest_own, round_own = stg.adjacent ? rest_own : step_own;
    if (b < 0) {
        t0 = (int64_t)blk * TILES;
        t1 = t0 + TILES;
        if (stg.tiles > 0 && t1 > tile0) t1 = tile0;
    } else if (own) {
        t0 = tile0 + tile_own;
        t1 = t0 + 1;
    } else {   // from the block that the last local tile belongs to
        const int64_t end = tile0 + stg.tiles, q = end / TILES + (b - own_blocks);
        t0 = q * TILES;
        t1 = t0 + TILES;
        if (t0 < end) t0 = end;
    }
    if (t1 > n_tiles) t1 = n_tiles;
    if (t0 >= t1) return;   // the whole block
    uint32_t n_chunks = 0;   // that may have handed edges over
    if (own && epoch[EPOCH_HANDED] == call_number(epoch)) {
        const int64_t all = (meta[META_EDGES] + EDGE_TILE - 1) / EDGE_TILE;
        n_chunks = (uint32_t)(all < stg.chunks ? all : stg.chunks);   // at most STAGE_EDGES_MAX / EDGE_TILE
    }
    const bool sums = n_chunks > 0;
    // The last `split` of a tile's blocks share its sums, the others leave (all but the last where nothing was handed over).
    uint32_t split = 1;
    if (sums) {
        split = n_chunks / (uint32_t)(SPLIT_MIN_EDGES / EDGE_TILE) / (uint32_t)stg.tiles;
        if (split > (uint32_t)stg.max_split) split = (uint32_t)stg.max_split;
        if (split < 1u) split = 1u;
    }
    const int share = own ? (int)round_own - (stg.max_split - (int)split) : 0;
    if (share < 0) return;
    if (own && share != (int)split - 1) {   // a share of a tile's sums: left for the block of the last share
        sum_handed_over(acc, stg, (int32_t)tile_own, n_chunks * share / split, n_chunks * (share + 1) / split);
        for (int i = threadIdx.x; i < CAND_TILE; i += CAND_PART_BLOCK) st_relaxed(&stg.part[(int64_t)b * CAND_TILE + i], acc[i]);
        wait_memory_ops();
        __syncthreads();
        if (threadIdx.x == 0) st_relaxed(&stg.part_flag[b], tag);
        return;
    }
    const int waves_per_tile = own ? WAVES : WAVES / TILES;
    const int64_t tile = own ? t0 : (t0 / TILES) * TILES + wave / waves_per_tile;   // of this wavefront
    const bool in_block = tile >= t0 && tile < t1;
    const int w_used = own ? CAND_WORDS / WAVES : W;   // words of this wavefront
    const uint32_t first_word = (uint32_t)((wave % waves_per_tile) * w_used);   // in the tile
    const int64_t word0 = tile * CAND_WORDS + first_word;
    const uint32_t tile_id = (uint32_t)tile * CAND_TILE;                         // below 2^31 + 1024
    const uint32_t lo_u = lo > 0 ? (uint32_t)lo : 0u, hi_u = hi > 0 ? (uint32_t)hi : 0u;
    uint64_t w[W];     // a lane's weights, ids ascending with (step, lane)
    uint32_t at[W];    // PACK: their ids' places in the tile,
    bool full[W];      // and whether that entry of the table goes back to zero
    int steps = w_used;
    if (!PACK || own) {
        uint64_t f8[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const bool have = in_block && k < w_used && word0 + k < n_words;
            f8[k] = have ? reinterpret_cast<const uint64_t *>(tileflag)[word0 + k] : 0ull;   // the word's eight group flags
        }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            if (PACK) at[k] = (first_word + k) * WAVE + lane;
            const uint32_t id = (uint32_t)(word0 + k) * 64u + lane;   // below 2^31 + 1024
            // only the touched groups of 8 ids (one 64-byte piece of the table each) are fetched
            w[k] = (((f8[k] >> (8 * (lane >> 3))) & 0xFFull) && id < (uint32_t)n_nodes) ? wtable[id] : 0ull;
        }
#pragma unroll
        for (int k = 0; k < W; ++k) full[k] = w[k] != 0;
    } else {
        // Lane l looks at the flag of the wavefront's l-th group of 8 ids; the touched ones, a quarter to a half of them in a
        // sparse neighbourhood, are then taken eight at a time, a lane per id.
        static_assert(!PACK || W * 8 == WAVE, "a lane per group");
        const int64_t group = word0 * 8 + lane;
        const bool touched = in_block && group < n_words * 8 && tileflag[in_block && group < n_words * 8 ? group : 0];
        const uint64_t mask = __ballot(touched), below = (1ull << lane) - 1ull;
        const int n_groups = __popcll(mask);
        const int to = touched ? __popcll(mask & below) : n_groups + __popcll(~mask & below);
        const int list = __builtin_amdgcn_ds_permute(to * 4, lane);   // lane r: the r-th touched group
        steps = (n_groups + 7) >> 3;
        // (no load under a condition: past the last touched group the first one is read again and dropped)
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const int r = k * 8 + (lane >> 3);
            at[k] = (first_word * 8 + (uint32_t)__shfl(list, r < n_groups ? r : 0, WAVE)) * 8 + (lane & 7);
            const uint32_t id = tile_id + at[k];
            full[k] = r < n_groups && id < (uint32_t)n_nodes;
            w[k] = wtable[id < (uint32_t)n_nodes ? id : (uint32_t)n_nodes - 1u];
        }
#pragma unroll
        for (int k = 0; k < W; ++k)
            if (!full[k]) w[k] = 0ull;   // (whole pieces go back to zero)
    }
    if (sums) {   // (what did not fit an entry, and ids of the tile outside the local range, have come through the table)
        sum_handed_over(acc, stg, (int32_t)tile_own, n_chunks * share / split, n_chunks);
        if (split > 1) {   // (the other shares' blocks were dispatched before and wait for nobody)
            const int64_t next = stg.adjacent ? 1 : stg.tiles, first = b - share * next;
            bool ok = true;
            if (threadIdx.x < (unsigned)share) ok = wait_tag(&stg.part_flag[first + threadIdx.x * next], tag, wait_limit(epoch));
            if (!ok) atomicOr(status, CSGS_ST_INTERNAL);
            __syncthreads();
            for (int i = threadIdx.x; i < CAND_TILE; i += CAND_PART_BLOCK) {
                unsigned long long v = acc[i];
                for (int k = 0; k < share; ++k) v += ld_relaxed(&stg.part[(first + k * next) * CAND_TILE + i]);
                acc[i] = v;
            }
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < CAND_WORDS / WAVES; ++k) {
            const uint32_t id = (uint32_t)(word0 + k) * 64u + lane;
            const unsigned long long v = acc[id - (uint32_t)(t0 * CAND_TILE)];
            if (v && id < hi_u) {
                w[k] += v;
                if (!PACK) {
                    wtable[id] = w[k];
                    tileflag[id >> 3] = 1;
                }
            }
        }
    }
    if (PACK && lane < W) *reinterpret_cast<uint64_t *>(&s_bits[PACK ? wave : 0][lane * 8]) = 0ull;
    {
        // counts from the ballots (scalar work), weights as the sum over everything and over the local ids: two
        // wave-wide 64-bit sums instead of three
        uint64_t cn = 0, wl = 0, wa = 0;   // cn packs (candidates << 32) | local candidates
#pragma unroll
        for (int k = 0; k < W; ++k) {
            if (PACK && k >= steps) continue;
            const uint32_t id = PACK ? tile_id + at[k] : (uint32_t)(word0 + k) * 64u + lane;
            const bool local = id >= lo_u && id < hi_u;
            cn += ((uint64_t)__popcll(__ballot(w[k] != 0)) << 32) | (uint64_t)__popcll(__ballot(w[k] != 0 && local));
            wa += w[k];
            wl += local ? w[k] : 0ull;
        }
        wl = wave_sum(wl); wa = wave_sum(wa);
        if (lane == 0) { lds[wave][0] = cn; lds[wave][1] = wl; lds[wave][2] = wa - wl; }
    }
    __syncthreads();
    // one wavefront publishes each tile; the block's last tile is the last wavefront's.
    // (packed count halves cannot carry: each is at most 1024 per tile)
    const int64_t t = t0 + wave;
    if (!PACK && t >= t1) return;
    if (t < t1) {
        const int w0 = own ? 0 : (int)(t % TILES) * waves_per_tile;
        unsigned long long mine = 0ull;
        if (lane < 3)
            for (int i = 0; i < waves_per_tile; ++i) mine += lds[w0 + i][lane];
        publish_tile(t, mine, partial, gtot);
    }
    if (!PACK || !in_block) return;
    // All of the tile's loads lie before the barrier above, and every entry of the table is written once: up to n_t by the weight
    // that belongs there, from there on by the lane that has read it.
    const int first_wave = wave - wave % waves_per_tile;
    uint32_t put = 0, n_t = 0;   // candidates before this wavefront's, and in the tile
    for (int i = 0; i < waves_per_tile; ++i) {
        const uint32_t n = (uint32_t)(lds[first_wave + i][0] >> 32);
        if (first_wave + i < wave) put += n;
        n_t += n;
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
        if (k >= steps) continue;
        const uint64_t word = __ballot(w[k] != 0);
        if (word) {
            if (w[k] != 0) wtable[tile_id + put + (uint32_t)__popcll(word & ((1ull << lane) - 1ull))] = w[k];
            const uint32_t bits = (uint32_t)(word >> (lane & ~7)) & 0xFFu;
            if ((lane & 7) == 0 && bits) s_bits[PACK ? wave : 0][(at[k] >> 3) - first_word * 8] = (uint8_t)bits;
            put += (uint32_t)__popcll(word);
        }
        if (full[k] && at[k] >= n_t) wtable[tile_id + at[k]] = 0ull;
    }
    if (lane < w_used && word0 + lane < n_words)
        reinterpret_cast<uint64_t *>(tileflag)[word0 + lane] = *reinterpret_cast<const uint64_t *>(&s_bits[PACK ? wave : 0][lane * 8]);
}

// The candidate sums after scan_wide, packed like cand_partials' packing kind: a block per bin (several for a local tile with many edges), whose groups
// it adds up in LDS, 64 runs at a time per wavefront, one per lane.  Bound by the latency of its loads -- where the groups lie, then
// the entries -- and by how many blocks a compute unit holds, so the first are asked for before anything else is known; before that, by vector
// instructions: 55 us for eight instances of 380 K edges with all eight wavefronts looking at every id, 41 with a bit per touched id.  (cand_partials
// after the narrow scan: 52; with the scan, 47 and 25.)
// FEW, several instances with up to BIN_FEW expected edges a bin and local tiles that take their share of them: a bin that is no local tile is one
// wavefront's if it has up to 512 entries.  The wavefront sets a bit for every id that an entry names, and an id's sum stands at the number of bits before it, so
// 512 sums do for 4096 ids, eight bins fit where one did, nothing waits at a barrier, and the sums are packed as they stand.  What holds more, or was met
// through the table, is the block's afterwards, one bin after the other; a block's bins lie far apart, as crowded ones lie side by side where ids follow the degree.  Eight
// instances of 380 K edges, 136 entries a bin: 39 -> 24 us (a block of 512 threads and 33 KB for each of 4488 bins took five and a half rounds).
// How many entries the local tiles take is known here only: with more than BIN_ONE_WAVE a bin left for the others these go one by one over the blocks that
// the device holds.  With scan, sums and emission of eight instances of 418 K edges, 745 a bin, 20 / 50 / 65 / 70 / 80 / 100 % of them remote, us:
//   a block per bin 91 / 92 / 92 / 93 / 93 / 90, wavefronts whatever they find 78 / 79 / 92 / 109 / 111 / 108, this 77 / 78 / 93 / 98 / 98 / 94
//   the remote ids by degree (density x^-2/3) 91 / 91 / 92 / 93 / 94 / 115, 118 / 155 / 175 / 180 / 191 / 210, 79 / 89 / 97 / 99 / 109 / 132
// (With blocks for every bin launched 83 at 20 %, as those that leave come in rounds too; bins of up to 2048 entries by a wavefront in several passes, or four wavefronts
// with room for 1024 sums each, cost the first column 1 to 3 us.)
template <bool WHOLE, bool FEW>   // WHOLE: as in scan_wide; FEW: a wavefront for each bin that is no local tile
__global__ __launch_bounds__(CAND_PART_BLOCK, 8) void bin_sums(uint64_t *__restrict__ wtable, uint8_t *__restrict__ tileflag, int64_t n_words, int64_t n_nodes,
                                                               int64_t n_tiles, int32_t lo, int32_t hi, const int64_t *__restrict__ meta, Stage stg,
                                                               const uint64_t *__restrict__ epoch, unsigned long long *__restrict__ partial, uint64_t *__restrict__ gtot,
                                                               int32_t *__restrict__ status, InstStride is)
{
    const InstBlock ib = inst_block(is, epoch[EPOCH_EVEN] != 0);
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block;
    constexpr int WAVES = CAND_PART_BLOCK / WAVE, U = 4;   // entries on their way per lane
    __shared__ unsigned long long acc[WIDE_IDS];
    __shared__ __attribute__((aligned(8))) uint32_t s_bits[WIDE_IDS / 32];   // ids with a weight
    __shared__ uint64_t lds[WAVES][3];
    __shared__ __attribute__((aligned(8))) uint32_t few_bits[FEW ? WAVES : 1][WIDE_IDS / 32];
    __shared__ int32_t crowded[WAVES], n_crowded, many_elsewhere;
    wtable = inst_ptr(wtable, is.ws); tileflag = inst_ptr(tileflag, is.ws); epoch = inst_ptr(epoch, is.ws);
    partial = inst_ptr(partial, is.ws); gtot = inst_ptr(gtot, is.ws);
    status = inst_ptr(status, is.buf); meta = inst_ptr(meta, is.ws);
    stg.e = inst_ptr(stg.e, is.ws); stg.off = inst_ptr(stg.off, is.ws);
    stg.part = inst_ptr(stg.part, is.ws); stg.part_flag = inst_ptr(stg.part_flag, is.ws);
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
    // blocks in the order of their bins, max_split for each of the local tiles (see cand_partials); FEW: the local tiles' before the others
    const int32_t own_blocks = stg.tiles * stg.max_split;
    auto whole_block = [&](int32_t b) {
        const bool own = b >= 0 && b < own_blocks;
        const uint32_t per_step = stg.adjacent ? (uint32_t)stg.max_split : (uint32_t)stg.tiles;
        const uint32_t step_own = own ? (uint32_t)b / per_step : 0u, rest_own = own ? (uint32_t)b % per_step : 0u;
        const uint32_t tile_own = stg.adjacent ? step_own : rest_own, round_own = stg.adjacent ? rest_own : step_own;
        const int32_t bin = b < 0 ? stg.below + b : (own ? stg.below + (int32_t)tile_own : stg.below + stg.tiles + (b - own_blocks));
        const int64_t most = stg.chunks / WIDE_CHUNKS;   // runs that the hand-over array holds, at least one
        const uint16_t *__restrict__ off = stg.off + bin;
        uint32_t beg, end;
        auto extents = [&](int64_t run) {   // where the bin's group lies in a run
            const uint16_t *p = off + (run < most ? run : 0) * WIDE_STRIDE;
            beg = p[0];
            end = p[1];
        };
        // share s takes the runs s, s + split, ...; of those, the first `readers` wavefronts one after the other (a bin's groups are
        // short: where there are few runs, fewer wavefronts have fewer instructions to issue)
        int readers = own ? WAVES : CAND_PART_TILES;
        extents(lane * readers + wave);
        const unsigned long long call = call_number(epoch), tag = call_tag(call, SLOT_CAND);
        int64_t n_chunks = 0, n_runs = 0;
        if (epoch[EPOCH_HANDED] == call) {
            n_chunks = (meta[META_EDGES] + EDGE_TILE - 1) / EDGE_TILE;
            n_runs = WHOLE ? (n_chunks + WIDE_CHUNKS - 1) / WIDE_CHUNKS : run_count(n_chunks, stg);
            if (n_runs > most) n_runs = most;
        }
        const bool table = epoch[EPOCH_ADDED] == call;   // something went through the table of accumulators
        const int64_t tile0 = stg.lo / CAND_TILE, local_end = tile0 + stg.tiles;
        int64_t t0, t1;
        if (b < 0) {
            t0 = (int64_t)(stg.below + b) * CAND_PART_TILES;
            t1 = t0 + CAND_PART_TILES;
            if (stg.tiles > 0 && t1 > tile0) t1 = tile0;
        } else if (own) {
            t0 = tile0 + tile_own;
            t1 = t0 + 1;
        } else {
            t0 = (local_end / CAND_PART_TILES + (b - own_blocks)) * CAND_PART_TILES;
            t1 = t0 + CAND_PART_TILES;
            if (t0 < local_end) t0 = local_end;
        }
        if (t1 > n_tiles) t1 = n_tiles;
        // the last `split` of a local tile's blocks share its sums, the others leave
        uint32_t split = 1;
        if (own && n_runs) {
            const int64_t want = (WHOLE ? n_runs * WIDE_CHUNKS : n_chunks) * EDGE_TILE / SPLIT_MIN_EDGES / stg.tiles;
            split = (uint32_t)(want < n_runs ? want : n_runs);
            if (split > (uint32_t)stg.max_split) split = (uint32_t)stg.max_split;
            if (split < 1u) split = 1u;
        }
        const int share = own ? (int)round_own - (stg.max_split - (int)split) : 0;
        if (t0 >= t1 || share < 0) return;   // the whole block
        const uint32_t ids = own ? CAND_TILE : WIDE_IDS;
        for (uint32_t i = tid; i < ids; i += CAND_PART_BLOCK) acc[i] = 0ull;
        for (uint32_t i = tid; i < ids / 32; i += CAND_PART_BLOCK) s_bits[i] = 0u;
        __syncthreads();
        const bool sparse = !own && n_runs <= CAND_PART_TILES * WAVE;   // few entries: their bits are set one by one, else from the sums
        if (split > 1 || (!own && !sparse)) {
            readers = WAVES;
            extents((int64_t)(lane * readers + wave) * split + share);
        }
        for (int64_t r0 = 0; r0 * split + share < n_runs && wave < readers; r0 += readers * WAVE) {
            const int64_t run = (r0 + lane * readers + wave) * split + share;
            // entry j of the sequence belongs to the first lane whose running count exceeds j
            const int32_t n = run < n_runs && beg <= end && end <= WIDE_EDGES ? (int32_t)(end - beg) : 0;
            const int32_t incl = wave_inclusive_scan<int32_t>(n);
            const int32_t total = __builtin_amdgcn_readlane(incl, WAVE - 1);
            const int32_t first = (int32_t)(run * WIDE_EDGES) + (int32_t)beg - (incl - n);   // it is entry first + j (at most STAGE_EDGES_MAX)
            extents((r0 + readers * WAVE + lane * readers + wave) * split + share);
            auto entry = [&](int32_t j) {
                int lo_l = 0, hi_l = WAVE - 1;
    #pragma unroll
                for (int it = 0; it < 6; ++it) {
                    const int mid = (lo_l + hi_l) >> 1;
                    if (__shfl(incl, mid, WAVE) > j) hi_l = mid; else lo_l = mid + 1;
                }
                const int32_t pos = __shfl(first, lo_l, WAVE) + j;
                return stg.e[j < total ? pos : 0];   // (unconditional; entry 0 stands in past the end)
            };
            auto take = [&](int32_t j, uint64_t v) {
                if (j >= total) return;
                const uint32_t at = (uint32_t)v & (ids - 1u);
                atomicAdd(&acc[at], (unsigned long long)(v / WIDE_IDS));
                if (sparse) atomicOr(&s_bits[at >> 5], 1u << (at & 31));
            };
            for (int32_t j0 = 0; j0 < total; j0 += U * WAVE) {
                if (total - j0 <= WAVE) {
                    take(j0 + lane, entry(j0 + lane));
                    break;
                }
                uint64_t v[U];
    #pragma unroll
                for (int u = 0; u < U; ++u) v[u] = entry(j0 + u * WAVE + lane);
    #pragma unroll
                for (int u = 0; u < U; ++u) take(j0 + u * WAVE + lane, v[u]);
            }
        }
        __syncthreads();
        if (own && share != (int)split - 1) {   // left for the block of the last share
            for (int i = tid; i < CAND_TILE; i += CAND_PART_BLOCK) st_relaxed(&stg.part[(int64_t)b * CAND_TILE + i], acc[i]);
            wait_memory_ops();
            __syncthreads();
            if (tid == 0) st_relaxed(&stg.part_flag[b], tag);
            return;
        }
        if (split > 1) {   // (the other shares' blocks were dispatched before and wait for nobody)
            const int64_t next = stg.adjacent ? 1 : stg.tiles, first = b - share * next;
            bool ok = true;
            if (tid < share) ok = wait_tag(&stg.part_flag[first + tid * next], tag, wait_limit(epoch));
            if (!ok) atomicOr(status, CSGS_ST_INTERNAL);
            __syncthreads();
            // (ids past the last node stay without a weight whatever a share holds that was not waited for: the weights go to the table side by side)
            const int n_ids = n_nodes - t0 * CAND_TILE < CAND_TILE ? (int)(n_nodes - t0 * CAND_TILE) : CAND_TILE;
            for (int i = tid; i < n_ids; i += CAND_PART_BLOCK) {
                unsigned long long v = acc[i];
                for (int k = 0; k < share; ++k) v += ld_relaxed(&stg.part[(first + k * next) * CAND_TILE + i]);
                acc[i] = v;
            }
            __syncthreads();
        }
        if (!sparse) {
            for (uint32_t i = tid; i < ids; i += CAND_PART_BLOCK) {
                const uint64_t word = __ballot(acc[i] != 0);
                if (lane == 0) reinterpret_cast<uint64_t *>(s_bits)[i >> 6] = word;
            }
            __syncthreads();
        }
        if (table) {   // what came through the table joins the sums, and the table is clean
            for (uint32_t i = tid; i < ids; i += CAND_PART_BLOCK) {
                const int64_t id = (own ? t0 : t0 / CAND_PART_TILES * CAND_PART_TILES) * CAND_TILE + i;
                if (id < t0 * CAND_TILE || id >= t1 * CAND_TILE || id >= n_nodes || !tileflag[id >> 3]) continue;
                const uint64_t more = wtable[id];
                if (!more) continue;
                wtable[id] = 0ull;
                acc[i] += more;
                atomicOr(&s_bits[i >> 5], 1u << (i & 31));
            }
            __syncthreads();
        }
        // Lane l looks at 16 ids of the wavefront's tile; a local tile is shared by all wavefronts, eight lanes' ids each.  The tile's weights go side by
        // side to the start of its piece of the table, and a bit per id in place of the groups' flags.
        if (!own && wave >= CAND_PART_TILES) return;
        const int64_t tile = own ? t0 : t0 / CAND_PART_TILES * CAND_PART_TILES + wave;
        if (tile < t0 || tile >= t1) return;   // (the whole wavefront; of a local tile, none)
        const uint32_t base = own ? 0u : (uint32_t)wave * CAND_TILE, tile_id = (uint32_t)tile * CAND_TILE;   // (ids: below 2^31 + 1024)
        const uint32_t piece = reinterpret_cast<const uint16_t *>(s_bits)[base / 16 + lane];
        const uint32_t cnt = (uint32_t)__popc(piece), incl = wave_inclusive_scan<uint32_t>(cnt), n_t = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
        const bool mine = !own || lane >> 3 == wave;
        const int64_t at16 = (int64_t)tile_id / 16 + lane;
        if (mine && at16 < n_words * 4 && (piece || table)) reinterpret_cast<uint16_t *>(tileflag)[at16] = (uint16_t)piece;
        const uint32_t id0 = tile_id + lane * 16;
        uint32_t put = tile_id + incl - cnt, n_local = 0;
        uint64_t wl = 0, wa = 0;
        for (uint32_t bits = mine ? piece : 0u; bits; bits &= bits - 1u) {
            const uint32_t k = (uint32_t)__ffs((int)bits) - 1u;
            const uint64_t v = acc[base + lane * 16 + k];
            wtable[put++] = v;
            const bool local = (int64_t)(id0 + k) >= lo && (int64_t)(id0 + k) < hi;
            wa += v;
            wl += local ? v : 0ull;
            n_local += local ? 1u : 0u;
        }
        wl = wave_sum(wl); wa = wave_sum(wa);
        n_local = wave_sum(n_local);
        if (own) {
            if (lane == 0) { lds[wave][0] = n_local; lds[wave][1] = wl; lds[wave][2] = wa - wl; }
            __syncthreads();   // (all wavefronts of a local tile's block come here)
            if (wave) return;
        }
        unsigned long long sum = lane == 0 ? (uint64_t)n_t << 32 | (own ? 0u : n_local) : (lane == 1 ? wl : wa - wl);
        if (own && lane < 3) {
            sum = lane == 0 ? (uint64_t)n_t << 32 : 0ull;
            for (int i = 0; i < WAVES; ++i) sum += lds[i][lane];
        }
        publish_tile(tile, sum, partial, gtot);
    };
    if constexpr (!FEW) {
        whole_block((int32_t)blk - stg.below);
    } else {
        if ((int32_t)blk < own_blocks) {
            whole_block((int32_t)blk);
            return;
        }
        const int32_t others = stg.bins - stg.tiles, groups = (others + WAVES - 1) / WAVES;
        const int32_t nth = (int32_t)blk - own_blocks < groups ? wave * groups + (int32_t)blk - own_blocks : others;
        const int32_t bin = nth < stg.below ? nth : nth + stg.tiles;
        const bool mine = nth < others;
        uint32_t beg = 0, end = 0;
        int32_t elsewhere = 0;   // entries of this lane's run that no local tile takes
        {
            const int64_t most = stg.chunks / WIDE_CHUNKS;
            const uint16_t *run = stg.off + (lane < most ? lane : 0) * WIDE_STRIDE, *p = run + (mine ? bin : 0);
            beg = p[0];
            end = p[1];
            if (wave == 0) elsewhere = (int32_t)run[stg.bins] - ((int32_t)run[stg.below + stg.tiles] - (int32_t)run[stg.below]);
        }
        const unsigned long long call = call_number(epoch);
        int64_t n_runs = 0;
        if (epoch[EPOCH_HANDED] == call) {
            n_runs = ((meta[META_EDGES] + EDGE_TILE - 1) / EDGE_TILE + WIDE_CHUNKS - 1) / WIDE_CHUNKS;
            const int64_t most = stg.chunks / WIDE_CHUNKS;
            if (n_runs > most) n_runs = most;
        }
        if (wave == 0) {
            elsewhere = wave_sum<int32_t>(lane < n_runs ? elsewhere : 0);
            if (lane == 0) {
                many_elsewhere = n_runs > WAVE || elsewhere > BIN_ONE_WAVE * others;   // (the same for all blocks)
                n_crowded = 0;
            }
        }
        __syncthreads();
        if (many_elsewhere) {
            for (int32_t i = (int32_t)blk - own_blocks; i < others; i += (int32_t)ib.blocks - own_blocks) {
                whole_block(i < stg.below ? i - stg.below : own_blocks + (i - stg.below));
                __syncthreads();
            }
            return;
        }
        if ((int32_t)blk - own_blocks >= groups) return;
        const int64_t tile0 = stg.lo / CAND_TILE, local_end = tile0 + stg.tiles;
        int64_t first_tile, t0, t1;
        if (nth < stg.below) {
            first_tile = t0 = (int64_t)nth * CAND_PART_TILES;
            t1 = t0 + CAND_PART_TILES;
            if (stg.tiles > 0 && t1 > tile0) t1 = tile0;
        } else {
            first_tile = t0 = (local_end / CAND_PART_TILES + (nth - stg.below)) * CAND_PART_TILES;
            t1 = t0 + CAND_PART_TILES;
            if (t0 < local_end) t0 = local_end;
        }
        if (t1 > n_tiles) t1 = n_tiles;
        constexpr int MOST = WIDE_IDS / WAVES;   // sums that a wavefront has room for
        const int64_t word = first_tile * CAND_WORDS + lane;   // this lane's 64 ids
        bool wave_does = mine && t0 < t1;
        if (wave_does && epoch[EPOCH_ADDED] == call)   // something went through the table of accumulators: of this bin?
            wave_does = !__any(first_tile + (lane >> 4) >= t0 && first_tile + (lane >> 4) < t1 && word < n_words && reinterpret_cast<const uint64_t *>(tileflag)[word < n_words ? word : 0] != 0ull);
        const int32_t n = lane < n_runs && beg <= end && end <= WIDE_EDGES ? (int32_t)(end - beg) : 0;
        const int32_t incl = wave_inclusive_scan<int32_t>(n);
        const int32_t total = __builtin_amdgcn_readlane(incl, WAVE - 1);
        if (mine && t0 < t1 && (!wave_does || total > MOST || n_runs > WAVE)) {   // the whole block's, afterwards
            if (lane == 0) crowded[atomicAdd(&n_crowded, 1)] = nth < stg.below ? nth - stg.below : own_blocks + (nth - stg.below);
            wave_does = false;
        }
        if (wave_does) {
            uint32_t *const bits = few_bits[FEW ? wave : 0];
            unsigned long long *const sum = acc + wave * MOST;
            reinterpret_cast<uint64_t *>(bits)[lane] = 0ull;
            // entry j of the sequence belongs to the first lane whose running count exceeds j
            const int32_t first = lane * WIDE_EDGES + (int32_t)beg - (incl - n);
            auto entry = [&](int32_t j) {
                int lo_l = 0, hi_l = WAVE - 1;
#pragma unroll
                for (int it = 0; it < 6; ++it) {
                    const int mid = (lo_l + hi_l) >> 1;
                    if (__shfl(incl, mid, WAVE) > j) hi_l = mid; else lo_l = mid + 1;
                }
                const int32_t pos = __shfl(first, lo_l, WAVE) + j;
                return stg.e[j < total ? pos : 0];
            };
            uint64_t v[MOST / WAVE];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = entry(u * WAVE + lane);
            if (total > U * WAVE) {
#pragma unroll
                for (int u = U; u < MOST / WAVE; ++u) v[u] = entry(u * WAVE + lane);
            } else {
#pragma unroll
                for (int u = U; u < MOST / WAVE; ++u) v[u] = 0ull;
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < MOST / WAVE; ++u) {
                const uint32_t at = (uint32_t)v[u] & (WIDE_IDS - 1u);
                if (u * WAVE + lane < total) atomicOr(&bits[at >> 5], 1u << (at & 31));
            }
            __builtin_amdgcn_wave_barrier();
            // a sum for every id that an entry names, in the order of the ids
            const uint64_t here = reinterpret_cast<const uint64_t *>(bits)[lane];
            const uint32_t cnt = (uint32_t)__popcll(here), upto = wave_inclusive_scan<uint32_t>(cnt), before = upto - cnt;
            const int32_t ids = (int32_t)__builtin_amdgcn_readlane((int)upto, WAVE - 1);
            for (int32_t i = lane; i < ids; i += WAVE) sum[i] = 0ull;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < MOST / WAVE; ++u) {
                if (u >= U && total <= U * WAVE) break;
                const uint32_t at = (uint32_t)v[u] & (WIDE_IDS - 1u);
                const uint32_t rank = (uint32_t)__shfl((int)before, (int)(at >> 6), WAVE);
                const uint64_t w = (uint64_t)(uint32_t)__shfl((int)(uint32_t)here, (int)(at >> 6), WAVE) |
                                   (uint64_t)(uint32_t)__shfl((int)(uint32_t)(here >> 32), (int)(at >> 6), WAVE) << 32;
                if (u * WAVE + lane < total)
                    atomicAdd(&sum[rank + (uint32_t)__popcll(w & ((1ull << (at & 63u)) - 1ull))], (unsigned long long)(v[u] / WIDE_IDS));
            }
            __builtin_amdgcn_wave_barrier();
            // out, each tile's to the start of its piece of the table; 16 lanes hold a tile
            const int64_t tile = first_tile + (lane >> 4);
            const uint32_t tile_id = (uint32_t)tile * CAND_TILE, tile_before = (uint32_t)__shfl((int)before, lane & 48, WAVE);
            if (here) reinterpret_cast<uint64_t *>(tileflag)[word] = here;
            uint32_t put = tile_id + before - tile_before, rank = before, n_local = 0;
            uint64_t wl = 0, wa = 0;
            for (uint64_t left = here; left; left &= left - 1ull) {
                const int64_t id = word * 64 + (__ffsll((unsigned long long)left) - 1);
                const uint64_t w = sum[rank++];
                wtable[put++] = w;
                const bool local = id >= lo && id < hi;
                wa += w;
                wl += local ? w : 0ull;
                n_local += local ? 1u : 0u;
            }
            uint64_t counts = (uint64_t)cnt << 32 | n_local;
#define CSGS_ROW_SUM(CTRL) (counts += dpp_move_t<uint64_t, CTRL, 0xF>(counts), wl += dpp_move_t<uint64_t, CTRL, 0xF>(wl), wa += dpp_move_t<uint64_t, CTRL, 0xF>(wa))
            CSGS_ROW_SUM(0x128); CSGS_ROW_SUM(0x124); CSGS_ROW_SUM(0x122); CSGS_ROW_SUM(0x121);   // row_ror: 16 lanes' sums, to all of them
#undef CSGS_ROW_SUM
            const int of = lane & 15;
            if (of < 3 && tile >= t0 && tile < t1) publish_sum(tile, of, of == 0 ? counts : (of == 1 ? wl : wa - wl), partial, gtot);
        }
        __syncthreads();
        const int32_t many = n_crowded;
        for (int32_t i = 0; i < many; ++i) {
            whole_block(crowded[i]);
            __syncthreads();
        }
    }
}

// Two kinds.  With PACKED a block takes four tiles (or two) that cand_partials has packed: where there are many tiles (several instances) the kernel is bound by
// vector instructions, and what they cost for the sums before a block, for the totals and for every 64-id word is then spent
// once for four tiles and on the candidates alone, while cand_partials takes longer (us per launch, cand_partials + this kernel, words / packed: 8 x 2392
// tiles with 65 candidates each 32 + 44 / 37 + 15, with 361 each 36 + 86 / 59 + 48; 1 x 9568 with 65 19 + 26 / 22 + 10, with 258 21 + 37 / 29 + 20; 8 x 1024
// with 501 19 + 42 / 26 + 33).  Below the line that depends on how full the tiles are, which the host does not know: few candidates are the quicker
// packed (1 x 2392 tiles with 65 each 8.1 + 11.2 / 9.7 + 5.4, 1 x 4784 12.9 + 15.5 / 15.2 + 7.2), many by words (1 x 2392 with 361 8.1 + 13.8 / 11.8 + 14.0,
// 1 x 1100 6.8 + 10.1 / 9.1 + 12.8).  From the line on no call was found that words serve better.
// (cand_partials at eight wavefronts per SIMD keeps two registers of the packing kind in scratch memory: its figures hold that.)
// After the wide scan of one instance two tiles a block: its local tiles are full and four of them many passes, one a block many blocks where there are many tiles
// (us, one / two / four: 2392 tiles, 710 K candidates 9.8 / 10.7 / 16.5, 213 K 7.0 / 9.4 / 14.6, 700 5.1 / 3.9 / 3.9; 9571 tiles, 772 K 19.8 / 12.8 / 17).
constexpr int EMIT_ONE = 2;
constexpr int64_t CAND_PACKED_FROM = 8192;   // tiles over all instances
template <bool PACKED, int TILES>
__global__ __launch_bounds__(256) void cand_emit(uint64_t *__restrict__ wtable, uint8_t *__restrict__ tileflag,
                                                 int64_t n_words, int64_t n_nodes, int64_t n_tiles, int32_t lo,
                                                 int32_t hi, SkewPolicy pol, const uint64_t *__restrict__ partial,
                                                 const uint64_t *__restrict__ gtot,
                                                 const int64_t *__restrict__ meta, int32_t shift_base,
                                                 uint64_t *__restrict__ epoch,
                                                 csgs_prob_stats *__restrict__ stats, int32_t *__restrict__ status,
                                                 int32_t *__restrict__ cand_id, uint64_t *__restrict__ cand_w,
                                                 uint64_t *__restrict__ cdf, float *__restrict__ q, int64_t cap, InstStride is)
{
    const InstBlock ib = inst_block(is, epoch[EPOCH_EVEN] != 0);
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block;
    __shared__ uint32_t s_cnt[4];
    static_assert(PACKED ? TILES <= 4 : TILES == 1, "a wavefront per packed tile");
    constexpr int WORDS = CAND_WORDS / 4;
    __shared__ uint32_t s_id[4][PACKED ? 1 : CAND_TILE / 4];    // the tile's candidates, packed: ids ...
    __shared__ uint64_t s_wt[4][PACKED ? 1 : CAND_TILE / 4];    // ... and fixed-point weights, per wavefront in id order
    __shared__ uint16_t s_at[4][PACKED ? CAND_TILE : 1];        // PACKED: places of a tile's candidates in it, in id order
    wtable = inst_ptr(wtable, is.ws); tileflag = inst_ptr(tileflag, is.ws); partial = inst_ptr(partial, is.ws);
    gtot = inst_ptr(gtot, is.ws); meta = inst_ptr(meta, is.ws); epoch = inst_ptr(epoch, is.ws);
    stats = inst_ptr(stats, is.buf); status = inst_ptr(status, is.buf); cand_id = inst_ptr(cand_id, is.buf);
    cand_w = inst_ptr(cand_w, is.buf); cdf = inst_ptr(cdf, is.buf); q = inst_ptr(q, is.buf);
    __shared__ uint64_t s_w[4];
    __shared__ uint64_t s_red[4][6];
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const int64_t t = (int64_t)blk * TILES;   // the block's first tile
    const int64_t g = t / 64, n_groups = (n_tiles + 63) / 64;
    // Loads are issued in the order flags, prefix inputs, accumulators, and consumed only after
    // all are in flight, so the tile's own data travels while the prefix is being summed.
    uint64_t flagged[WORDS];   // the eight group flags of each 64-id word (one byte per 8 ids)
    const int64_t bits_at = t * (CAND_TILE / 16) + threadIdx.x;   // PACKED: a lane holds the bits of 16 ids
    uint32_t bits = 0;
    if (PACKED) {
        if (wave < TILES && bits_at < n_words * 4) bits = reinterpret_cast<const uint16_t *>(tileflag)[bits_at];
    } else {
#pragma unroll
        for (int k = 0; k < WORDS; ++k) {
            const int64_t word_idx = t * CAND_WORDS + wave * WORDS + k;
            flagged[k] = word_idx < n_words ? reinterpret_cast<const uint64_t *>(tileflag)[word_idx] : 0ull;
        }
    }
    // sums over everything (tot) and over what lies before this tile (pre): group sums before my
    // group, then tile sums before me inside my group
    uint64_t gv[3] = {0, 0, 0}, pv[3] = {0, 0, 0};
    if ((int64_t)threadIdx.x < n_groups) {
#pragma unroll
        for (int i = 0; i < 3; ++i) gv[i] = gtot[(int64_t)threadIdx.x * 4 + i];
    }
    {
        const int64_t j = g * 64 + threadIdx.x;
        if (threadIdx.x < 64 && j < t) {
#pragma unroll
            for (int i = 0; i < 3; ++i) pv[i] = partial[j * 4 + i];
        }
    }
    uint64_t w[WORDS];
    if (PACKED) {
        if (bits) reinterpret_cast<uint16_t *>(tileflag)[bits_at] = 0;   // back to the clean state
        const uint32_t n = (uint32_t)__popc(bits), incl = wave_inclusive_scan<uint32_t>(n);
        if (lane == WAVE - 1) s_cnt[wave] = incl;
        uint16_t *list = s_at[wave] + (incl - n);
        for (; bits; bits &= bits - 1u) *list++ = (uint16_t)(lane * 16 + __ffs(bits) - 1);
    } else {
#pragma unroll
        for (int k = 0; k < WORDS; ++k) {
            // node ids are below 2^31 and a tile adds at most 1023: 32-bit arithmetic, half the instructions
            const uint32_t id = ((uint32_t)t * CAND_WORDS + wave * WORDS + k) * 64u + lane;
            w[k] = (((flagged[k] >> (8 * (lane >> 3))) & 0xFFull) && id < (uint32_t)n_nodes) ? wtable[id] : 0ull;
        }
    }
    uint64_t tot[3], pre[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        tot[i] = gv[i];
        pre[i] = ((int64_t)threadIdx.x < g ? gv[i] : 0ull) + pv[i];
    }
    for (int64_t j = (int64_t)threadIdx.x + blockDim.x; j < n_groups; j += blockDim.x) {  // more than 256 groups
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint64_t v = gtot[j * 4 + i];
            tot[i] += v;
            if (j < g) pre[i] += v;
        }
    }
    // group j's sums are held by thread j and the in-group tile sums by the first 64 threads: with fewer
    // than 64 groups only the first wavefront has anything to add up (the others hold zeros)
    if ((int64_t)wave * WAVE < n_groups) {
#pragma unroll
        for (int i = 0; i < 3; ++i) { tot[i] = wave_sum(tot[i]); pre[i] = wave_sum(pre[i]); }
    }
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) { s_red[wave][i] = tot[i]; s_red[wave][3 + i] = pre[i]; }
    }
    __syncthreads();
    uint32_t c0 = 0, c1 = 0, c2 = 0, n_t = 0;   // candidates of the first wavefront's piece, of the first two, ..., of the block
    auto counts = [&]() {
        c0 = s_cnt[0];
        c1 = c0 + s_cnt[1];
        c2 = c1 + s_cnt[2];
        n_t = c2 + s_cnt[3];
    };
    // A pass takes ROWS times 256 candidates, a wavefront up to ROWS rows of 64 that lie one after the other (as many for each wavefront as the pass needs).
    // Four where the tiles are few and full: one distribution of 65 536 rows 66.8 -> 65.0 us.  In their registers fewer blocks fit, so one where there are
    // many (step of eight mini-batches 662 -> 669 with four, level with two) and where the list lies in LDS.
    constexpr int ROWS = PACKED && TILES == EMIT_ONE ? 4 : 1;
    uint32_t id[ROWS];
    uint64_t wi[ROWS];
    auto rows_of = [&](uint32_t base) { return n_t - base > 256u * (ROWS - 1) ? (uint32_t)ROWS : (n_t - base + 255u) / 256u; };
    auto place = [&](uint32_t base, uint32_t rows, int r) { return base + ((uint32_t)wave * rows + (uint32_t)r) * WAVE + (uint32_t)lane; };
    auto fetch = [&](uint32_t base) {   // candidates of the block, the last one in the place of those that do not exist
        const uint32_t rows = rows_of(base);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if ((uint32_t)r >= rows) break;
            const uint32_t at = place(base, rows, r), i = at < n_t ? at : n_t - 1u;
            if (ROWS == 1 && at >= n_t) break;   // (one row: nothing waits for this load before it is used)
            const int src = i < c0 ? 0 : (i < c1 ? 1 : (i < c2 ? 2 : 3));
            const uint32_t k = i - (src == 0 ? 0u : (src == 1 ? c0 : (src == 2 ? c1 : c2)));
            if (PACKED) {
                const uint32_t first = ((uint32_t)t + src) * CAND_TILE;
                id[r] = first + s_at[src][k];
                wi[r] = wtable[first + k];
                if (ROWS == 1) wtable[first + k] = 0ull;   // back to the clean state
            } else {
                id[r] = s_id[src][k];
                wi[r] = s_wt[src][k];
            }
        }
    };
    if (PACKED) {   // the first pass' weights are asked for before the sums are put together
        counts();
        if (n_t) fetch(0);
    }
    {   // lanes 0 .. 5 add up one of the six sums each; the others get them by lane broadcast (not every lane all 24 terms)
        const uint64_t mine = lane < 6 ? s_red[0][lane] + s_red[1][lane] + s_red[2][lane] + s_red[3][lane] : 0ull;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            tot[i] = __shfl(mine, i, WAVE);
            pre[i] = __shfl(mine, 3 + i, WAVE);
        }
    }
    const uint64_t n_cand = tot[0] >> 32, n_local = tot[0] & 0xFFFFFFFFull;
    uint64_t m_local, m_remote;
    resolve_skew(pol, n_cand, n_cand - n_local, &m_local, &m_remote);
    const uint64_t total_w = tot[1] * m_local + tot[2] * m_remote;
    const double total_d = (double)total_w;

    // The tile's candidates (about one id in fifteen in a sparse neighbourhood) are first packed into LDS, every
    // wavefront its own four words in id order, the accumulators and flags going back to their clean state on the way.
    // Everything that costs instructions per candidate -- the skewed weight, the 64-bit running sum, q, the five
    // stores -- is then done on the packed list, by as many wavefronts as it fills, with contiguous stores.
    if (!PACKED) {
        uint32_t my_cnt = 0;
#pragma unroll
        for (int k = 0; k < WORDS; ++k) {
            const int slot = wave * (WORDS) + k;
            const uint32_t my_id = ((uint32_t)t * CAND_WORDS + slot) * 64u + lane;
            const uint64_t word = __ballot(w[k] != 0);
            if (w[k] != 0) {
                const uint32_t at = my_cnt + (uint32_t)__popcll(word & ((1ull << lane) - 1ull));
                s_id[wave][at] = my_id;
                s_wt[wave][at] = w[k];
                wtable[my_id] = 0ull;  // back to the clean state
            }
            my_cnt += (uint32_t)__popcll(word);
            if (flagged[k] && lane == 0) reinterpret_cast<uint64_t *>(tileflag)[t * CAND_WORDS + slot] = 0ull;  // back to the clean state
        }
        if (lane == 0) s_cnt[wave] = my_cnt;
        __syncthreads();
        counts();
    }
    const uint32_t lo_u = lo > 0 ? (uint32_t)lo : 0u, hi_u = hi > 0 ? (uint32_t)hi : 0u;
    const int64_t base_cnt = (int64_t)(pre[0] >> 32);
    uint64_t run_w = pre[1] * m_local + pre[2] * m_remote;   // skewed weight before the packed candidate at pass_base
    for (uint32_t pass_base = 0; pass_base < n_t; pass_base += ROWS * 256u) {
        const uint32_t rows = rows_of(pass_base);
        if (!PACKED || pass_base) fetch(pass_base);
        uint64_t wsk[ROWS], incl[ROWS], sum = 0;   // sum: of this wavefront's candidates
        if (place(pass_base, rows, 0) - (uint32_t)lane < n_t) {   // (the whole wavefront)
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                if ((uint32_t)r >= rows) break;
                const uint32_t i = place(pass_base, rows, r);
                wsk[r] = i < n_t ? wi[r] * ((id[r] >= lo_u && id[r] < hi_u) ? m_local : m_remote) : 0ull;
                incl[r] = sum + wave_inclusive_scan(wsk[r]);
                sum = ROWS == 1 ? incl[r] : __shfl(incl[r], WAVE - 1, WAVE);
            }
        }
        if (lane == WAVE - 1) s_w[wave] = sum;
        __syncthreads();
        uint64_t before = run_w;
        for (int w2 = 0; w2 < wave; ++w2) before += s_w[w2];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if ((uint32_t)r >= rows) break;
            const uint32_t i = place(pass_base, rows, r);
            if (i >= n_t) break;
            if (PACKED && ROWS > 1) {   // back to the clean state, now that all weights of the pass are on their way
                const int src = i < c0 ? 0 : (i < c1 ? 1 : (i < c2 ? 2 : 3));
                wtable[((uint32_t)t + src) * CAND_TILE + i - (src == 0 ? 0u : (src == 1 ? c0 : (src == 2 ? c1 : c2)))] = 0ull;
            }
            const int64_t pos = base_cnt + i;
            if (pos < cap) {
                cand_id[pos] = (int32_t)id[r];
                cand_w[pos] = wi[r];
                cdf[pos] = before + incl[r];
                if (q) q[pos] = (float)((double)wsk[r] / total_d);
            }
        }
        run_w += s_w[0] + s_w[1] + s_w[2] + s_w[3];
        __syncthreads();   // s_w is written again in the next pass
    }
    if (t + TILES >= n_tiles && threadIdx.x == 0) {
        stats->n_cand = (int64_t)n_cand;
        stats->n_local = (int64_t)n_local;
        stats->n_remote = (int64_t)(n_cand - n_local);
        stats->w_local = tot[1];
        stats->w_remote = tot[2];
        stats->total = total_w;
        stats->shift = shift_for_rows(shift_base, meta[META_ROWS]);
        stats->edges_scanned = meta[META_EDGES_TRUE];
        stats->skew_fx = (int32_t)m_local * (m_remote ? 1 : -1);
        int32_t st = 0;
        if (n_cand == 0 || total_w == 0) st |= CSGS_ST_EMPTY_CANDIDATES;
        if ((int64_t)n_cand > cap) st |= CSGS_ST_CAND_OVERFLOW;
        if (st) atomicOr(status, st);
        epoch[EPOCH_CALLS] += 1ull;  // last kernel of the call; no block of this kernel reads the counter
    }
}

__global__ void fill_zero(uint64_t *p, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0ull;
}

static int ceil_log2_u64(uint64_t n)
{
    int e = 0;
    while (e < 63 && (1ull << e) < n) ++e;
    return e;
}

// 61 - ceil(log2 s_fx) - ceil(log2 rmax): the fraction bits a single row could use
static int shift_base_for(int64_t s_fx, float rownorm2_max)
{
    int e_r = 0;
    while (e_r < 64 && ldexp(1.0, e_r) < (double)rownorm2_max) ++e_r;
    return 61 - ceil_log2_u64((uint64_t)s_fx) - e_r;
}

}  // namespace csgs

int csgs::launch_row_prefix(const int64_t *rowptr, int64_t n_nodes, const int32_t *S, int32_t nS, const int32_t *nS_dev,
                            const Workspace &w, const RowOffsets &rows, int32_t *status, hipStream_t st)
{
    const unsigned tiles = (unsigned)(((int64_t)nS + ROW_TILE - 1) / ROW_TILE);
    CSGS_LAUNCH(K_ROW_PREFIX, row_prefix, dim3(tiles, 1, (unsigned)w.n_inst), dim3(256), st, rowptr, n_nodes, S, nS, nS_dev,
                w.epoch, w.rp_ts, w.rp_tiles, rows.eoff, rows.rowstart, rows.meta, w.chunk_cap * EDGE_TILE, rows.bound_note, status,
                inst_stride(w));
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

using namespace csgs;

extern "C" size_t csgs_workspace_bytes(int64_t n_nodes, int32_t nS_max, int32_t B_max, int64_t edges_max)
{
    if (n_nodes <= 0 || n_nodes > 0x7FFFFFFFll || nS_max <= 0 || B_max <= 0 || edges_max <= 0) return 0;
    return carve(nullptr, n_nodes, nS_max, B_max, edges_max).bytes;
}

extern "C" size_t csgs_workspace_clean_bytes(int64_t n_nodes)
{
    if (n_nodes <= 0) return 0;
    return carve(nullptr, n_nodes, 1, 1, 1).clean_bytes;
}

extern "C" int csgs_workspace_init(csgs_workspace *ws, void *stream)
{
    if (!ws) return CSGS_EINVAL;
    ws->rows_buf = 0;
    ws->has_draw = 0;
    ws->has_next = 0;
    ws->draw_B = 0;
    Workspace w;
    const int rc = open_workspace(ws, ws->n_nodes, 1, 1, &w);
    if (rc != CSGS_OK) return rc;
    const size_t n = w.bytes * (size_t)w.n_inst / 8;
    const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    CSGS_LAUNCH(K_FILL_ZERO, fill_zero, dim3(blocks), dim3(256), (hipStream_t)stream, (uint64_t *)ws->base, n);
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

namespace csgs {
// one block per instance
__global__ void set_word(uint64_t *p, uint64_t v, int64_t stride) { *(uint64_t *)((char *)p + (int64_t)blockIdx.x * stride) = v; }
}  // namespace csgs

extern "C" int csgs_workspace_wait_limit(csgs_workspace *ws, int64_t polls, void *stream)
{
    if (!ws) return CSGS_EINVAL;
    Workspace w;
    const int rc = open_workspace(ws, ws->n_nodes, 1, 1, &w);
    if (rc != CSGS_OK) return rc;
    const uint64_t v = polls < 0 ? 0ull : (uint64_t)(polls > 0x7FFFFFF0ll ? 0x7FFFFFF0ll : polls) + 1ull;
    CSGS_LAUNCH(K_FILL_ZERO, csgs::set_word, dim3((unsigned)w.n_inst), dim3(1), (hipStream_t)stream, w.epoch + EPOCH_WAIT, v,
                (int64_t)w.bytes);
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

// Fixed-point parameters.  shift = min(52, 61 - ceil(log2 nS) - ceil(log2 s_fx) - ceil(log2 rmax)):
// the skewed total is at most nS * rmax * 2^shift * s_fx plus rounding slack, below 2^63.
extern "C" int csgs_fixed_point(int32_t nS, float skew, float rownorm2_max, int32_t *shift, int64_t *s_fx)
{
    if (nS <= 0 || !(skew >= 1.0f) || skew > 1048576.0f || !(rownorm2_max > 0.0f) || !isfinite(rownorm2_max))
        return CSGS_EINVAL;
    const int64_t sfx = llround((double)skew * 16.0);
    int sh = shift_base_for(sfx, rownorm2_max) - ceil_log2_u64((uint64_t)nS);
    if (sh > 52) sh = 52;
    if (shift) *shift = sh;
    if (s_fx) *s_fx = sfx;
    return sh < 24 ? CSGS_ERANGE : CSGS_OK;
}

static int build_probs_impl(const csgs_graph *g, const int32_t *S, int32_t nS, const int32_t *nS_dev,
                            float shift_skew, SkewPolicy pol,
                            int32_t *cand_id, uint64_t *cand_w, uint64_t *cdf, float *q, int64_t cap,
                            csgs_prob_stats *stats, csgs_workspace *ws, int32_t *status, void *stream)
{
    if (!g || !g->rowptr || !g->colidx || !g->val || g->n_nodes <= 0 || g->n_nodes > 0x7FFFFFFFll ||
        g->local_lo > g->local_hi || nS <= 0 || !cand_id || !cand_w || !cdf || cap <= 0 || !stats || !ws || !status)
        return CSGS_EINVAL;
    // S == NULL: the rows are the node set of the latest csgs_sample_layer on this workspace, whose
    // offsets that call has prepared; nS must be its capacity (the B of that draw)
    if (ws->scan_mode < 0 || ws->scan_mode > 2) return CSGS_EINVAL;
    const bool chained = S == nullptr;
    if (chained && (!ws->has_next || nS_dev || nS != ws->draw_B)) return CSGS_EINVAL;
    int32_t shift;
    int64_t s_fx;
    int rc = csgs_fixed_point(nS, shift_skew, g->rownorm2_max, &shift, &s_fx);
    if (rc != CSGS_OK) return rc;
    if (pol.mode == 0) pol.s_fx = (uint64_t)s_fx;
    if (pol.mode == 1) pol.s_fx_max = (uint64_t)s_fx;
    Workspace w;
    rc = open_workspace(ws, g->n_nodes, nS, 1, &w);
    if (rc != CSGS_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int64_t n_words = (g->n_nodes + 63) / 64;

    // the shift for nS rows has passed the range check; fewer rows on the device only widen it
    const int32_t shift_base = shift_base_for(s_fx, g->rownorm2_max);
    if (chained) {
        ws->rows_buf ^= 1;      // the set the adjacency pass prepared
    } else {
        rc = launch_row_prefix(g->rowptr, g->n_nodes, S, nS, nS_dev, w, w.rows[ws->rows_buf & 1], status, st);
        if (rc != CSGS_OK) return rc;
    }
    ws->has_next = 0;
    const RowOffsets &rows = w.rows[ws->rows_buf & 1];
    // The number of edges is known on the device only: rows of the graph's mean degree are a guess that hubs can exceed many
    // times over.  What depends on the number is decided on the device, and there are never fewer blocks than the device
    // holds (those without a chunk leave at once) unless the workspace describes fewer chunks.  With several instances the
    // least is a block per compute unit over all of them: there, blocks that leave are not free (eight instances of 14
    // chunks, 32 blocks each 12 us, 64 blocks 14, 256 blocks 28).
    // (us for scan and sums, grid and hand-over by the mean degree / as here: 256 rows of 5000 edges, mean degree 8, 270 / 68;
    // the 1024 rows of most edges in 2.4 M, 6.4 M edges of them, 336 / 282.)
    const double mean = (double)nS * ((double)g->nnz / (double)g->n_nodes) / EDGE_TILE, guess = mean * 1.25 + 16.0;
    int64_t chunks = guess < (double)SCAN_GRID ? (int64_t)guess : SCAN_GRID;
    const int64_t least = w.n_inst == 1 ? SCAN_GRID : SCAN_GRID / 8 / w.n_inst;
    if (chunks < least) chunks = least;
    if (chunks > w.chunk_cap) chunks = w.chunk_cap;
    // tiles that meet the local id range, when the hand-over can cover them and is wanted
    const bool range_ok = g->local_hi > g->local_lo && g->local_lo >= 0 && g->local_hi <= g->n_nodes;
    const int64_t tile0 = range_ok ? g->local_lo / CAND_TILE : 0, tile1 = range_ok ? ((int64_t)g->local_hi - 1) / CAND_TILE + 1 : 0;
    const int32_t min_chunks = ws->scan_mode == 2 ? 0 : HAND_OVER_MIN_CHUNKS;
    // With several instances the blocks that a hand-over needs are launched only where it is to be expected (eight instances of
    // 13 chunks and 114 local tiles, the sums without / with them 14.4 / 16.6 us); rows that hold more go through atomics there.
    const bool hand = ws->scan_mode != 1 && (w.n_inst == 1 ? (double)w.chunk_cap : mean * w.n_inst) >= (double)min_chunks;
    const int32_t tiles = (hand && tile1 - tile0 <= SUB_MAX) ? (int32_t)(tile1 - tile0) : 0;
    // Blocks per tile: what the expected chunks can use, and in case the rows hold more, a block per compute unit in all with
    // one instance.  (Not as many as there might ever be use for: 150 idle ones cost a launch 1 us.)  Blocks of a tile that all
    // have work lie side by side, an XCD taking the same chunks of all tiles (6.8 K chunks, 64 tiles 28 us, else 32); those of
    // which some may leave do not, as the ones that stay would be on a few XCDs only.
    int64_t split = 1;
    bool adjacent = true;
    if (tiles) {
        const int64_t each = (int64_t)tiles * w.n_inst;
        split = (int64_t)fmin(mean, (double)w.stage_chunks) * EDGE_TILE / tiles / SPLIT_MIN_EDGES;
        if (w.n_inst == 1 && split < SPLIT_BLOCKS / 2 / tiles) {
            split = SPLIT_BLOCKS / 2 / tiles;
            adjacent = false;
        }
        if (split > SPLIT_BLOCKS / each) split = SPLIT_BLOCKS / each;
        if (split > w.split_blocks / tiles) split = w.split_blocks / tiles;
        if (split > WAVE) split = WAVE;
        if (split < 1) split = 1;
    }
    const int64_t per = w.n_inst == 1 && w.n_tiles <= CAND_PART_ONE ? 1 : CAND_PART_TILES;
    const int64_t below = tiles ? (tile0 + per - 1) / per : 0;
    const int64_t rest = tiles ? (w.n_tiles + per - 1) / per - tile1 / per : (w.n_tiles + per - 1) / per;   // blocks of `per` tiles past the local ones
    const int64_t part_blocks = below + tiles * split + rest;
    const bool wide = ws->scan_mode == 0 && per == CAND_PART_TILES && w.stage_chunks >= WIDE_CHUNKS && below + tiles + rest <= WIDE_BINS &&
                      (below + rest) * w.n_inst >= WIDE_MIN_BINS &&
                      fmin(mean, (double)w.chunk_cap) * w.n_inst >= (double)(tiles ? WIDE_MIN_CHUNKS : WIDE_MIN_CHUNKS_NARROW_OFF);
    const Stage stg{w.stage, w.stage_off, w.stage_chunks, range_ok ? g->local_lo : 0, range_ok ? g->local_hi : 0, tiles, (int32_t)split,
                    adjacent ? 1 : 0, w.n_inst, min_chunks, (int32_t)(tiles ? below : rest), (int32_t)(below + tiles + rest),
                    (int32_t)(w.n_inst == 1 ? (w.stage_chunks / WIDE_CHUNKS < WIDE_RUNS ? w.stage_chunks / WIDE_CHUNKS : WIDE_RUNS) : 0), (unsigned long long *)w.split_sum, (unsigned long long *)w.split_flag,
                    w.gtot, (w.n_tiles + 63) / 64 * 4};
    if (wide) {
        int64_t runs = (int64_t)(guess < 1e9 ? guess : 1e9) / WIDE_CHUNKS + 1;
        if (runs < 256 && w.n_inst == 1) runs = 256;
        if (runs > SCAN_GRID / 4) runs = SCAN_GRID / 4;
        if (runs > (w.chunk_cap + WIDE_CHUNKS - 1) / WIDE_CHUNKS) runs = (w.chunk_cap + WIDE_CHUNKS - 1) / WIDE_CHUNKS;
        const InstGrid ig = inst_grid(w, runs, WIDE_BLOCK);
#define CSGS_SCAN_WIDE(WHOLE)                                                                                                                    \
    CSGS_LAUNCH(K_SCAN_EDGES, scan_wide<WHOLE>, ig.grid, dim3(WIDE_BLOCK), st, g->colidx, g->val, g->n_nodes, g->nnz, shift_base, rows.meta, \
                w.chunk_cap * EDGE_TILE, rows.eoff, rows.rowstart, w.wtable, w.tileflag, rows.bound_note, w.epoch, status, stg, ig.is)
        if (stg.runs) CSGS_SCAN_WIDE(false); else CSGS_SCAN_WIDE(true);
#undef CSGS_SCAN_WIDE
    } else {
        const InstGrid ig = inst_grid(w, chunks, 256);
        CSGS_LAUNCH(K_SCAN_EDGES, scan_edges, ig.grid, dim3(256), st, g->colidx, g->val,
                    g->n_nodes, g->nnz, shift_base, rows.meta, w.chunk_cap * EDGE_TILE, rows.eoff, rows.rowstart, w.wtable,
                    w.tileflag, rows.bound_note, w.epoch, status, stg, ig.is);
    }
    CSGS_LAUNCH_CHECK();
    const int64_t others = below + rest;
    const bool few = wide && !stg.runs && tiles && fmin(mean, (double)w.chunk_cap) * EDGE_TILE <= (double)(BIN_FEW * others);
    // FEW: a wavefront for every other bin, and, should they be taken one by one, as many blocks as the device holds (else these leave at once)
    constexpr int64_t FEW_BINS = CAND_PART_BLOCK / WAVE, FEW_BLOCKS = SCAN_GRID / 2;
    int64_t few_blocks = (others + FEW_BINS - 1) / FEW_BINS;
    if (few_blocks < FEW_BLOCKS / w.n_inst) few_blocks = FEW_BLOCKS / w.n_inst < others ? FEW_BLOCKS / w.n_inst : others;
    const InstGrid part = inst_grid(w, few ? tiles * split + few_blocks : part_blocks, CAND_PART_BLOCK);
#define CSGS_CAND_PARTIALS(TILES, PACK)                                                                                                       \
    CSGS_LAUNCH(K_CAND_PARTIALS, (cand_partials<TILES, PACK>), part.grid, dim3(CAND_PART_BLOCK), st, w.wtable, w.tileflag, n_words, g->n_nodes, \
                w.n_tiles, g->local_lo, g->local_hi, rows.meta, stg, (int32_t)(tiles ? below : part_blocks), w.epoch,                   \
                (unsigned long long *)w.partial, w.gtot, status, part.is)
    const bool packed = wide || w.n_tiles * w.n_inst >= CAND_PACKED_FROM;   // (then `per` is CAND_PART_TILES)
#define CSGS_BIN_SUMS(WHOLE, FEW)                                                                                                             \
    CSGS_LAUNCH(K_CAND_PARTIALS, (bin_sums<WHOLE, FEW>), part.grid, dim3(CAND_PART_BLOCK), st, w.wtable, w.tileflag, n_words, g->n_nodes, w.n_tiles, \
                g->local_lo, g->local_hi, rows.meta, stg, w.epoch, (unsigned long long *)w.partial, w.gtot, status, part.is)
    if (wide && stg.runs) CSGS_BIN_SUMS(false, false);
    else if (few) CSGS_BIN_SUMS(true, true);
    else if (wide) CSGS_BIN_SUMS(true, false);
    else if (packed) CSGS_CAND_PARTIALS(CAND_PART_TILES, true);
    else if (per == 1) CSGS_CAND_PARTIALS(1, false);
    else CSGS_CAND_PARTIALS(CAND_PART_TILES, false);
#undef CSGS_CAND_PARTIALS
#undef CSGS_BIN_SUMS
    CSGS_LAUNCH_CHECK();
    const int64_t emit_tiles = !packed ? 1 : (wide && w.n_inst == 1 ? EMIT_ONE : 4);
    const InstGrid emit = inst_grid(w, (w.n_tiles + emit_tiles - 1) / emit_tiles, 256);
#define CSGS_CAND_EMIT(PACKED, TILES)                                                                                                       \
    CSGS_LAUNCH(K_CAND_EMIT, (cand_emit<PACKED, TILES>), emit.grid, dim3(256), st, w.wtable, \
                w.tileflag, n_words, g->n_nodes, w.n_tiles, g->local_lo, g->local_hi, pol, w.partial, w.gtot, rows.meta, shift_base, w.epoch, \
                stats, status, cand_id, cand_w, cdf, q, cap, emit.is)
    if (emit_tiles == 4) CSGS_CAND_EMIT(true, 4); else if (packed) CSGS_CAND_EMIT(true, EMIT_ONE); else CSGS_CAND_EMIT(false, 1);
#undef CSGS_CAND_EMIT
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

extern "C" int csgs_build_probs(const csgs_graph *g, const int32_t *S, int32_t nS, const int32_t *nS_dev, float skew,
                                int32_t *cand_id,
                                uint64_t *cand_w, uint64_t *cdf, float *q, int64_t cap, csgs_prob_stats *stats,
                                csgs_workspace *ws, int32_t *status, void *stream)
{
    SkewPolicy pol = {0, 0, 0.0, 0, 0};
    float shift_skew = skew;
    if (isinf(skew) && skew > 0) {   // "Local" version: remote candidates get probability zero
        pol.mode = 2;
        shift_skew = 1.0f;
    }
    return build_probs_impl(g, S, nS, nS_dev, shift_skew, pol, cand_id, cand_w, cdf, q, cap, stats, ws, status, stream);
}

extern "C" int csgs_build_probs_auto(const csgs_graph *g, const int32_t *S, int32_t nS, const int32_t *nS_dev, float D,
                                     int32_t B,
                                     float skew_max, int32_t *cand_id, uint64_t *cand_w, uint64_t *cdf, float *q,
                                     int64_t cap, csgs_prob_stats *stats, csgs_workspace *ws, int32_t *status,
                                     void *stream)
{
    if (!(D >= 0.0f) || !isfinite(D) || B <= 0) return CSGS_EINVAL;
    SkewPolicy pol = {1, 0, (double)D, (int64_t)B, 0};
    return build_probs_impl(g, S, nS, nS_dev, skew_max, pol, cand_id, cand_w, cdf, q, cap, stats, ws, status, stream);
}
