// Shared device helpers and the workspace layout of the csgs library (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <type_traits>
#include "csgs.h"
#include "profile.hpp"

namespace csgs {

constexpr int WAVE = 64;

typedef double doublex4 __attribute__((ext_vector_type(4)));   // what a lane holds of a 16 x 16 tile of sums

#define CSGS_LAUNCH_CHECK()                                   \
    do {                                                      \
        if (hipGetLastError() != hipSuccess) return CSGS_ELAUNCH; \
    } while (0)

__host__ __device__ inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---------------------------------------------------------------- workspace
// "clean" sections are all-zero between calls and come first.  The per-edge sections come
// last; how many edges they can hold follows from the size the caller passed.
constexpr int CAND_TILE = 1024;   // node ids per block in the candidate scan
constexpr int EDGE_TILE = 1024;   // edges per chunk in the flat edge passes
constexpr int SCAN_GRID = 2048;   // most chunk blocks of the weight scan (grid-stride over chunks, they wait for nobody): more than the device holds at once
constexpr int HIT_MIN_WORDS = 16;     // fewest 64-position bitmap words a block of the hit compaction takes
constexpr int HIT_GRID = 512;         // most blocks of it
constexpr int64_t HIT_COUNT_WORDS = 49152;   // most bitmap words of which every block counts those before its own itself
constexpr int ROW_TILE = 1024;    // rows of S per block in the degree prefix
// Hand-over of the weight scan: edges that end in the local id range are left, chunk by chunk, for blocks that each add
// up one tile of CAND_TILE ids in LDS.
constexpr int SUB_MAX = 320;                      // most such tiles: local ranges up to 319 K ids
constexpr int SUB_STRIDE = SUB_MAX + 32;          // entries per chunk of the groups' begins: SUB_MAX + 1, in whole 64-byte pieces
constexpr int64_t SPLIT_BLOCKS = 512;             // most blocks of a launch over which the local tiles are split
constexpr int64_t STAGE_EDGES_MAX = 8ll << 20;    // most edges of a call that are handed over this way (the others go through atomics)
constexpr int EPOCH_WORDS = 16;       // counters on the device (lookback.hpp)
constexpr int META_WORDS = 4;
constexpr int META_ROWS = 0;          // rows the latest row_prefix covered (the count behind eoff / rowstart)
constexpr int META_EDGES = 1;         // eoff[rows]: edges of those rows (0 when above the workspace's capacity)
constexpr int META_EDGES_TRUE = 2;    // their true number

// Words of workspace a single-pass scan over at most `tiles` tiles with nv sums per tile needs
// (one tag word and nv sums per tile, and twice that per group of 64 tiles).
__host__ __device__ constexpr size_t scan_state_words(int64_t tiles, int nv)
{
    return (size_t)(1 + nv) * (size_t)(tiles + 2 * (tiles / 64 + 2));
}
static_assert(HIT_COUNT_WORDS * 64 / CAND_TILE >= (int64_t)scan_state_words(HIT_GRID, 1), "the hit compaction's scan state in hit_ts");

struct RowOffsets {
    int64_t *eoff;       // [nS + 1] exclusive prefix of the degrees of the rows
    int64_t *rowstart;   // [nS + 1] rowptr[S[a]]
    int64_t *meta;       // [META_WORDS] resolved on the device: row count, edge count, true edge count
    int2 *bound_note;    // [chunk_cap + 2] for the edge position t * EDGE_TILE: (first row of a chunk that starts there, first row
                         // whose offset is at or beyond it), left by the row pass for the edge passes
};

struct Workspace {
    // clean: all-zero whenever no call is in flight
    uint64_t *wtable;    // [n_nodes]  per-node fixed-point weight accumulator
    uint8_t *tileflag;   // [8 * ceil(n_nodes/64)] byte g = 1: some node of ids 8g .. 8g+7 was touched (read 8 at a time: one 64-id word; between the two candidate kernels of a packed call: a bit per id)
    uint32_t *hit;       // [n_nodes]  draws per candidate position
    // persistent: zeroed once, then never cleared; an entry counts only if it carries the tag of
    // the current call
    uint64_t *rank;      // [n_nodes]  (tag << 32) | (position in S_next + 1)
    uint64_t *member;    // [(n_nodes + 31) / 32]  (tag << 32) | one bit per id of the word's 32: in S_next of the draw with that tag
    uint64_t *partial;   // [4 * n_tiles] per-tile candidate counts and weight sums
    uint64_t *gtot;      // [4 * ceil(n_tiles / 64)] the same per group of 64 tiles
    uint64_t *hit_ts;    // [n_tiles] in a draw with a long position bitmap the scan state of the hit compaction
    uint64_t *epoch;     // [EPOCH_WORDS] call counter and draw tag (see lookback.hpp); advanced on the device
    uint64_t *cbitmap[2]; // [ceil(n_nodes/64)] bit set = candidate position was drawn.  Draws take turns: the compaction of one
                         // clears what the one before set
    // per call.  The row offsets exist twice: while the adjacency pass of one layer reads one set,
    // its spare blocks prepare the other for the next layer (rows = the node set just sampled).
    RowOffsets rows[2];
    uint64_t *adj_ts;    // scan state of the edge chunks (1 sum per chunk of 1024 edges)
    uint32_t *adj_cnt;   // [chunk_cap] kept edges of every edge chunk | 1 << 31 when a row starts at the chunk's first edge
    uint64_t *rp_ts;     // scan state of the row tiles (1 sum per tile of ROW_TILE rows)
    double *pdbl;        // [B]      inclusion probabilities in double
    // hand-over of local-range edges from the weight scan to the candidate sums; `stage` also takes the kept edges of a
    // chunk (column | value << 32) from the adjacency's marking pass to its placing pass
    uint64_t *stage;     // [stage_chunks * EDGE_TILE] weight and id of a handed-over edge; a chunk's edges lie grouped by tile
    uint16_t *stage_off; // [stage_chunks * SUB_STRIDE] per chunk and local tile: where its group begins (and the previous one ends)
    uint64_t *split_sum; // [split_blocks * CAND_TILE] and tags: sums of the blocks that share a local tile
    uint64_t *split_flag;// [split_blocks] persistent
    int64_t split_blocks;
    int64_t stage_chunks;
    int64_t chunk_cap;   // chunks of EDGE_TILE edges the adjacency scan can describe
    int64_t n_tiles, rp_tiles;
    size_t clean_bytes;  // size of the clean part
    size_t bytes;        // size of one instance's workspace (a multiple of 256)
    int32_t n_inst;      // instances a call on this workspace processes (set by open_workspace)
    int64_t buf_stride;  // bytes between consecutive instances' caller buffers
};

// Several independent instances of a call run in the same launches, and every per-instance pointer moves by that
// instance's stride in bytes -- `ws` for what lives in the workspace (instance k's workspace follows instance
// k - 1's), `buf` for the caller's arrays.  The graph is shared.  With one instance nothing moves.
// Blocks come instance after instance (blockIdx.z selects it), or the instances in turn (inst_grid() below).
struct InstStride {
    int64_t ws, buf;
    int32_t n;   // instances of a one-dimensional grid; 0: blockIdx.z is the instance
};
// The strides of instance k, for inst_ptr().
__device__ inline InstStride at_instance(const InstStride &is, int64_t k) { return InstStride{is.ws * k, is.buf * k, is.n}; }
__device__ inline InstStride at_instance(const InstStride &is) { return at_instance(is, blockIdx.z); }
// Instance of this block, its number among the instance's, and how many those are.
struct InstBlock {
    uint32_t k, block, blocks;
};
__device__ inline InstBlock inst_block(const InstStride &is, bool in_turn)
{
    if (!is.n) return InstBlock{blockIdx.z, blockIdx.x, gridDim.x};
    const uint32_t n = (uint32_t)is.n, each = gridDim.x / n;
    return in_turn ? InstBlock{blockIdx.x % n, blockIdx.x / n, each} : InstBlock{blockIdx.x / each, blockIdx.x % each, each};
}
// In turn as well, but moved on by one with every turn, so that no XCD is an instance's own.
__device__ inline InstBlock inst_block_spread(const InstStride &is)
{
    if (!is.n) return InstBlock{blockIdx.z, blockIdx.x, gridDim.x};
    const uint32_t n = (uint32_t)is.n, b = blockIdx.x / n;
    return InstBlock{(blockIdx.x + b) % n, b, gridDim.x / n};
}
template <typename T>
__device__ inline T *inst_ptr(T *p, int64_t bytes)
{
    // (pointer arithmetic, not integer arithmetic: the result is still known to point to global memory, so loads
    // through it are global loads and not the slower flat ones)
    return p ? (T *)((char *)const_cast<typename std::remove_const<T>::type *>(p) + bytes) : p;   // null stays null
}
constexpr int MAX_INSTANCES = 64;

// The same for the layer compute calls, whose arrays come in four groups with a stride each.
struct CompStride {
    int64_t adj;   // what the sampling calls wrote: adjacency arrays, row counts, source-row map, id lists
    int64_t x;     // the input matrix (0: one table shared by all instances)
    int64_t xr;    // staged remote rows
    int64_t out;   // the output matrix
};
// A pointer of this block's instance; the compute kernels take an instance after the other.
template <typename T>
__device__ inline T *comp_ptr(T *p, int64_t stride)
{
    return p ? (T *)((char *)const_cast<typename std::remove_const<T>::type *>(p) + (int64_t)blockIdx.z * stride) : p;
}
struct CompInst {
    int32_t n = 1;
    CompStride cs = {0, 0, 0, 0};
};
// Checks a caller's csgs_inst_strides (null: one instance).
__host__ inline int open_instances(const csgs_inst_strides *d, CompInst *out)
{
    *out = CompInst{};
    if (!d) return CSGS_OK;
    if (d->n_inst < 1 || d->n_inst > MAX_INSTANCES || d->adj < 0 || d->x < 0 || d->x_remote < 0 || d->out < 0 ||
        ((d->adj | d->x | d->x_remote | d->out) & 15))
        return CSGS_EINVAL;
    out->n = d->n_inst;
    out->cs = CompStride{d->adj, d->x, d->x_remote, d->out};
    return CSGS_OK;
}

// Layout of a workspace sized for (n_nodes, nS_max, B_max, edges_max).  Every call carves with the
// same four numbers (they travel in the caller's csgs_workspace descriptor), so the persistent
// parts never move.
__host__ inline Workspace carve(void *base, int64_t n_nodes, int64_t nS_max, int64_t B_max, int64_t edges_max)
{
    Workspace w;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return (char *)base + o;
    };
    const size_t words = (size_t)(n_nodes + 63) / 64;
    w.n_tiles = (n_nodes + CAND_TILE - 1) / CAND_TILE;
    w.chunk_cap = (edges_max + EDGE_TILE - 1) / EDGE_TILE;
    if (w.chunk_cap < 1) w.chunk_cap = 1;
    w.wtable = (uint64_t *)take((size_t)n_nodes * 8);
    w.tileflag = (uint8_t *)take(words * 8);
    w.hit = (uint32_t *)take((size_t)n_nodes * 4);
    w.clean_bytes = off;
    w.rank = (uint64_t *)take((size_t)n_nodes * 8);
    w.member = (uint64_t *)take((size_t)((n_nodes + 31) / 32) * 8);
    w.partial = (uint64_t *)take((size_t)w.n_tiles * 4 * 8);
    w.gtot = (uint64_t *)take((size_t)((w.n_tiles + 63) / 64) * 4 * 8);
    w.hit_ts = (uint64_t *)take((size_t)w.n_tiles * 8);
    w.epoch = (uint64_t *)take(EPOCH_WORDS * 8);
    for (int b = 0; b < 2; ++b) w.cbitmap[b] = (uint64_t *)take(words * 8);
    w.adj_ts = (uint64_t *)take(scan_state_words(w.chunk_cap, 1) * 8);
    w.adj_cnt = (uint32_t *)take((size_t)w.chunk_cap * 4);
    w.rp_tiles = (nS_max + ROW_TILE - 1) / ROW_TILE;
    w.rp_ts = (uint64_t *)take(scan_state_words(w.rp_tiles, 1) * 8);
    for (int b = 0; b < 2; ++b) {
        w.rows[b].eoff = (int64_t *)take((size_t)(nS_max + 1) * 8);
        w.rows[b].rowstart = (int64_t *)take((size_t)(nS_max + 1) * 8);
        w.rows[b].meta = (int64_t *)take(META_WORDS * 8);
        w.rows[b].bound_note = (int2 *)take((size_t)(w.chunk_cap + 2) * sizeof(int2));
    }
    w.pdbl = (double *)take((size_t)B_max * 8);
    w.stage_chunks = w.chunk_cap < STAGE_EDGES_MAX / EDGE_TILE ? w.chunk_cap : STAGE_EDGES_MAX / EDGE_TILE;
    w.stage = (uint64_t *)take((size_t)w.stage_chunks * EDGE_TILE * 8);
    w.stage_off = (uint16_t *)take((size_t)w.stage_chunks * SUB_STRIDE * 2);
    w.split_blocks = w.n_tiles * (w.stage_chunks / 64 + 1);
    if (w.split_blocks > SPLIT_BLOCKS) w.split_blocks = SPLIT_BLOCKS;
    w.split_sum = (uint64_t *)take((size_t)w.split_blocks * CAND_TILE * 8);
    w.split_flag = (uint64_t *)take((size_t)w.split_blocks * 8);
    w.bytes = off;
    w.n_inst = 1;
    w.buf_stride = 0;
    return w;
}

// Checks a descriptor against a call's sizes and carves it.  Returns CSGS_OK or an error code.
__host__ inline int open_workspace(csgs_workspace *d, int64_t n_nodes, int64_t nS, int64_t B, Workspace *out)
{
    if (!d || !d->base || ((uintptr_t)d->base & 255) || d->n_nodes != n_nodes || d->nS_max <= 0 || d->B_max <= 0 ||
        d->edges_max <= 0)
        return CSGS_EINVAL;
    if (nS > d->nS_max || B > d->B_max) return CSGS_EWORKSPACE;
    const int32_t n_inst = d->n_inst > 1 ? d->n_inst : 1;
    if (n_inst > MAX_INSTANCES || (n_inst > 1 && (d->inst_stride <= 0 || (d->inst_stride & 255)))) return CSGS_EINVAL;
    *out = carve(d->base, d->n_nodes, d->nS_max, d->B_max, d->edges_max);
    out->n_inst = n_inst;
    out->buf_stride = n_inst > 1 ? d->inst_stride : 0;
    return out->bytes * (size_t)n_inst <= d->bytes ? CSGS_OK : CSGS_EWORKSPACE;
}

__host__ inline InstStride inst_stride(const Workspace &w) { return InstStride{(int64_t)w.bytes, w.buf_stride, 0}; }
// Grid of `blocks` blocks per instance for kernels that take the instances in turn: block b of instance k is the (b n + k)-th of all.  The hardware deals
// consecutive blocks round-robin to the 8 XCDs, so an instance's blocks stay on one XCD of eight instances, two of four, four of two, and so do the tables they look
// things up in, which one L2 then holds.  A launch then lasts as long as its largest instance on its part of the device; kernels whose work follows
// from the rows' edges do so only where those are about even, as the weight scan has noted (the note is the same for all blocks of a launch).  Only for kernels whose blocks wait for nobody or for lower blocks of their
// instance (those were dispatched before them): not for resident grids, see below.  An odd number of instances would spread over the XCDs either way.
// (us per launch, after each other / in turn, eight instances of 8192 rows of 51 edges: marking pass of the adjacency 26.9 / 22.8, emission 24.4 / 19.6, draws 15.8 / 13.2,
// compaction 12.4 / 10.4, candidate sums 39.2 / 38.5, sampling of a layer 163 / 148; two instances 86 / 85, four 119 / 111, six 138 / 129, sixteen 299 / 273.  One instance of
// 32768 rows and seven of 2048 in turn 274, after each other 168, as noted 174.  The placing pass wins nothing and goes after each other.  The weight scan looks nothing up
// and its blocks fill a compute unit: level alone, 1 to 2 % of a step with another stream's products beside it (bench, eight instances: 81.5 after each other, 79.6 in turn), so
// inst_block_spread(), which costs 60 for 43 with one instance of 32768 rows and seven of 8192 and is level with 2048; in turn 78.)
struct InstGrid {
    dim3 grid;
    InstStride is;
};
__host__ inline InstGrid inst_grid(const Workspace &w, int64_t blocks, int threads)
{
    InstStride is = inst_stride(w);
    if (w.n_inst % 2 || blocks * w.n_inst * threads > 0x7FFFFFFFll) return InstGrid{dim3((unsigned)blocks, 1, (unsigned)w.n_inst), is};
    is.n = w.n_inst;
    return InstGrid{dim3((unsigned)(blocks * w.n_inst)), is};
}
__host__ inline dim3 each_instance(const Workspace &w, int64_t blocks) { return dim3((unsigned)blocks, 1, (unsigned)w.n_inst); }

// Grid of a kernel whose blocks wait for each other and stride over a tile count known only on
// the device: of the blocks of 256 threads that a compute unit holds (by threads, registers and LDS),
// resident_grid(per_cu), a share.  Such a kernel must have all its blocks resident at once.  Alone on the device that is
// certain.  Beside kernels of other streams it still holds as long as the waiting kernels in flight fit
// together, because every other kernel drains by itself: the one-pass adjacency filter (72 registers, 13 KB of LDS:
// seven blocks per unit) launches a quarter of what the device holds, so CALL_SEQUENCES on as many workspaces
// can be in flight on one device.  That is the documented limit.
constexpr int CALL_SEQUENCES = 4;
// With several instances per call (blockIdx.z) the grid of such a kernel is that many times as large, but blocks
// wait only for blocks of their own instance and the hardware hands out a grid's blocks in
// ascending x, then y, then z: an instance is dispatched completely before the next one starts, a
// completely dispatched instance finishes by itself and frees its places, and at most one instance
// per kernel is ever partly dispatched -- so what must fit at once is still one instance per
// waiting kernel in flight.
__host__ inline int resident_grid(int per_cu)
{
    static std::atomic<int> cached[64];   // compute units per device, 0 = not asked yet (zero-initialised)
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 32 * per_cu;
    int cus = cached[dev].load(std::memory_order_relaxed);
    if (cus == 0) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 32;
        cached[dev].store(cus, std::memory_order_relaxed);   // every thread would store the same value
    }
    return per_cu * cus;
}

// Degrees of the rows S, their exclusive prefix and CSR starts into `rows`.  The row count is
// min(*nS_dev, nS) when nS_dev is given; the kernel leaves it, and the edge count, in rows.meta for
// the kernels that follow.  Defined with the weight scan.
int launch_row_prefix(const int64_t *rowptr, int64_t n_nodes, const int32_t *S, int32_t nS, const int32_t *nS_dev,
                      const Workspace &w, const RowOffsets &rows, int32_t *status, hipStream_t st);

// A row count given on the host (n) or, when n_dev is not null, on the device with n as its bound.
__device__ inline int32_t resolve_count(int32_t n, const int32_t *__restrict__ n_dev)
{
    if (!n_dev) return n;
    const int32_t d = *n_dev;
    return d < 0 ? 0 : (d < n ? d : n);
}

// ---------------------------------------------------------------- wave helpers
__device__ inline int lane_id() { return (int)(threadIdx.x & (WAVE - 1)); }

// Lane exchanges of the wave-wide scan run on the data-parallel-primitive path of the vector ALU
// (no LDS round trip): shifts by 1, 2, 4, 8 inside each row of 16 lanes with zero fill, then lane
// 15 of a row broadcast to the next row (rows 1 and 3), then lane 31 to rows 2 and 3.
template <int CTRL, int ROW_MASK>
__device__ inline uint32_t dpp_move(uint32_t v)
{
    // old = 0: lanes outside ROW_MASK, and lanes whose source falls outside the row, receive 0
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, true);
}

template <typename T, int CTRL, int ROW_MASK>
__device__ inline T dpp_move_t(T v)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit integers");
    if (sizeof(T) == 4) return (T)dpp_move<CTRL, ROW_MASK>((uint32_t)v);
    const uint64_t x = (uint64_t)v;
    const uint32_t lo = dpp_move<CTRL, ROW_MASK>((uint32_t)x), hi = dpp_move<CTRL, ROW_MASK>((uint32_t)(x >> 32));
    return (T)(((uint64_t)hi << 32) | lo);
}

// The scan of a 64-bit value held as two halves.  A step is v += (v moved by the step's pattern), as an add with carry
// whose first operand comes through the DPP path -- two instructions, where a moved copy (two moves, each with its
// zero fill) and a 64-bit add take five.  Lanes the pattern leaves out are not written and keep v, which is what adding
// the zero fill gave.  The carry travels in VCC.  Two wait states lie between a vector instruction that writes VCC and
// one that reads it, and between one that writes a register and a DPP read of it; inside an asm statement the compiler
// does not count them.  With the s_nop between the two halves of a step, the next step's reads are far enough behind.
#define CSGS_SCAN_STEP64(PATTERN)                         \
    "v_add_co_u32_dpp %0, vcc, %0, %0 " PATTERN "\n\t"      \
    "s_nop 1\n\t"                                         \
    "v_addc_co_u32_dpp %1, vcc, %1, %1, vcc " PATTERN "\n\t"
__device__ inline uint64_t wave_inclusive_scan64(uint64_t v)
{
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    asm volatile("s_nop 1\n\t"
                 CSGS_SCAN_STEP64("row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1")
                 CSGS_SCAN_STEP64("row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1")
                 CSGS_SCAN_STEP64("row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:1")
                 CSGS_SCAN_STEP64("row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:1")
                 CSGS_SCAN_STEP64("row_bcast:15 row_mask:0xa bank_mask:0xf")
                 CSGS_SCAN_STEP64("row_bcast:31 row_mask:0xc bank_mask:0xf")
                 : "+v"(lo), "+v"(hi)
                 :
                 : "vcc");
    return ((uint64_t)hi << 32) | lo;
}

template <typename T>
__device__ inline T wave_inclusive_scan(T v)
{
    if (sizeof(T) == 8) return (T)wave_inclusive_scan64((uint64_t)v);
    v += dpp_move_t<T, 0x111, 0xF>(v);  // row_shr:1
    v += dpp_move_t<T, 0x112, 0xF>(v);  // row_shr:2
    v += dpp_move_t<T, 0x114, 0xF>(v);  // row_shr:4
    v += dpp_move_t<T, 0x118, 0xF>(v);  // row_shr:8
    v += dpp_move_t<T, 0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_move_t<T, 0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Sum over the wavefront, the same value in every lane.
template <typename T>
__device__ inline T wave_sum(T v)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit integers");
    const T s = wave_inclusive_scan(v);
    if (sizeof(T) == 4) return (T)__builtin_amdgcn_readlane((int)s, WAVE - 1);
    const uint64_t x = (uint64_t)s;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, WAVE - 1);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), WAVE - 1);
    return (T)(((uint64_t)hi << 32) | lo);
}

// Exclusive scan over the threads of a block (blockDim.x a multiple of 64, at most 1024).
// Returns the exclusive prefix; *block_total receives the sum over the block.
template <typename T>
__device__ inline T block_exclusive_scan(T v, T *lds /*[17]*/, T *block_total)
{
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const int nwaves = (int)(blockDim.x >> 6);
    T incl = wave_inclusive_scan(v);
    __syncthreads();  // lds may still be read from a previous use
    if (lane == WAVE - 1) lds[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        T t = lane < nwaves ? lds[lane] : T(0);
        T s = wave_inclusive_scan(t);
        if (lane < nwaves) lds[lane] = s - t;
        if (lane == nwaves - 1) lds[16] = s;
    }
    __syncthreads();
    *block_total = lds[16];
    return incl - v + lds[wave];
}

// First indices in [0, n) with a[idx] >= key[i], found by the whole wavefront: every round the 64 lanes
// probe the ends of 64 equal segments at once, so an array of 8192 entries takes 3 dependent loads
// instead of 13, and the searches for several keys go through their rounds together.  All lanes must call it
// with the same arguments; all get the results.
template <int K, typename T, typename I>
__device__ inline void wave_lower_bounds(const T *__restrict__ a, I n, const T (&key)[K], I (&out)[K])
{
    const int lane = lane_id();
    I lo[K], hi[K];
    bool more = false;
#pragma unroll
    for (int i = 0; i < K; ++i) { lo[i] = 0; hi[i] = n; more = more || n > 0; }
    while (more) {
        T v[K];
        I step[K];
        bool probe[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const I len = hi[i] - lo[i];
            step[i] = (len + WAVE - 1) / WAVE;
            const I seg_end = lo[i] + ((lane + 1) * step[i] < len ? (lane + 1) * step[i] : len);  // exclusive
            const I seg_beg = lo[i] + (lane * step[i] < len ? lane * step[i] : len);
            probe[i] = seg_end > seg_beg;
            v[i] = a[probe[i] ? seg_end - 1 : 0];
        }
        more = false;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (hi[i] <= lo[i]) continue;   // found
            const I len = hi[i] - lo[i];
            // empty segments sit past the end: treat as "all remaining entries are >= key"
            const uint64_t m = __ballot(probe[i] ? v[i] >= key[i] : true);
            const int first = m ? __ffsll((unsigned long long)m) - 1 : WAVE;
            const I fb = lo[i] + (first * step[i] < len ? first * step[i] : len);
            const I fe = lo[i] + ((first + 1) * step[i] < len ? (first + 1) * step[i] : len);
            if (fe <= fb) {             // no segment ends at or above key: every entry is below it
                lo[i] = hi[i];
            } else if (step[i] == 1) {  // segments are single entries: entry fb is the first >= key
                lo[i] = fb;
                hi[i] = fb;
            } else {                    // a[fe - 1] >= key and everything before fb is below key
                lo[i] = fb;
                hi[i] = fe;
            }
            more = more || hi[i] > lo[i];
        }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) out[i] = lo[i];
}

// ---------------------------------------------------------------- flat edge chunks
// The edges of the rows of S, concatenated in row order, form one sequence of E edges; position
// e belongs to the row a with eoff[a] <= e < eoff[a+1] and sits at rowstart[a] + (e - eoff[a])
// in the CSR arrays.  A block works on chunks of consecutive positions, so the work per block does
// not depend on the degree distribution.
//
// Which row a position belongs to: the rows that overlap a chunk set the bit of the position where they start (a row
// that began before the chunk: position 0) and leave there what must be added to a position to get its CSR address.  A position's row is
// the one of the last bit at or before it: the 64 positions of a word are a wavefront's lanes, so that is a mask and a count of leading
// zeros, and the last bit before a word comes from one scan over the words.  Empty rows set no bit.  (us, a binary search per edge over
// the rows staged in LDS / this: weight scan of 2.3 K edges 8.8 / 5.8, of 52 K 11 / 8.3, of eight times 380 K 52 / 47; marking pass of the adjacency
// 28.7 / 26.0 for the eight, 65 / 59 for 6.7 M; its one-pass form 11.8 / 7.9 for 2.3 K and 10.3 / 8.0 for 52 K.)
template <int TILE>
struct EdgeMap {
    static constexpr int WORDS = TILE / WAVE;
    static_assert(WORDS <= WAVE, "a lane per word");
    int64_t delta[TILE];          // at a row's first position: CSR address minus position
    unsigned long long starts[WORDS];
};

// What the row pass left for the chunk boundaries (see row_prefix_tile): the chunk of edge positions [t0 * EDGE_TILE, t1 * EDGE_TILE)
// is covered by the rows [first, end).
struct ChunkRows {
    int32_t first, end;
};
__device__ inline ChunkRows chunk_rows(const int2 *__restrict__ bound, int64_t t0, int64_t t1)
{
    const ChunkRows r{bound[t0].x, bound[t1].y};
    return ChunkRows{t0 == 0 ? 0 : r.first, r.end};
}

// Row r.first + threadIdx.x: where its edges begin and end in the flat order, and in the CSR arrays.  (Loads without a condition: a row that
// does not exist reads another one's.)  nS > 0.
struct RowEdges {
    int64_t beg, end, csr;
};
__device__ inline RowEdges row_edges(const int64_t *__restrict__ eoff, const int64_t *__restrict__ rowstart, int32_t nS, int64_t a)
{
    if (a > nS - 1) a = nS - 1;   // (also after a prefix broken by a failed wait)
    if (a < 0) a = 0;
    return RowEdges{eoff[a], eoff[a + 1], rowstart[a]};
}
__device__ inline RowEdges first_rows(const int64_t *__restrict__ eoff, const int64_t *__restrict__ rowstart, int32_t nS, const ChunkRows &r)
{
    return row_edges(eoff, rowstart, nS, (int64_t)r.first + threadIdx.x);
}

// Rows of a chunk per thread from which its positions are searched for in the rows one by one instead of the rows walked through: nearly all
// of them are empty then (1 M rows of which the last 10 K have 50 edges each: weight scan 1252 us walked through, 33 searched; 200 K rows, the last 10 K of 20 edges 234 and 18).
constexpr int32_t MAP_ROWS = 32;   // by the searches that a thread has on their way
// Fills `m` for the edge positions [c0, c0 + len).  Called by all threads of the block, with its first_rows().  Returns where row
// r.first + threadIdx.x starts, relative to c0 (the caller's place for that row's pointer).
template <int TILE>
__device__ inline int32_t map_edges(EdgeMap<TILE> &m, const int64_t *__restrict__ eoff, const int64_t *__restrict__ rowstart, int32_t nS,
                                    int64_t c0, int32_t len, ChunkRows &r, RowEdges row)
{
    if (r.first < 0) r.first = 0;   // (a prefix broken by a failed wait)
    if (r.end > nS) r.end = nS;
    __syncthreads();   // the previous chunk's readers are done
    if (threadIdx.x < EdgeMap<TILE>::WORDS) m.starts[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) m.delta[0] = 0;
    __syncthreads();
    const int64_t off = row.beg - c0;
    constexpr int AT_ONCE = TILE > EDGE_TILE ? 1 : 2;   // searches on their way (the scan of many edges has no registers to spare)
    if (r.end - r.first > MAP_ROWS / AT_ONCE * (int32_t)blockDim.x) {
        for (int32_t x0 = (int32_t)threadIdx.x; x0 < len; x0 += AT_ONCE * (int32_t)blockDim.x) {
            int32_t lo[AT_ONCE], hi[AT_ONCE], x[AT_ONCE];
            bool more = false;
#pragma unroll
            for (int k = 0; k < AT_ONCE; ++k) {
                lo[k] = r.first;
                hi[k] = r.end;
                x[k] = x0 + k * (int32_t)blockDim.x;
                if (x[k] >= len) x[k] = x0;
            }
            do {   // eoff[lo] <= c0 + x < eoff[hi]
                more = false;
#pragma unroll
                for (int k = 0; k < AT_ONCE; ++k) {
                    const int32_t mid = lo[k] + (hi[k] - lo[k]) / 2;
                    if (eoff[mid] - c0 <= (int64_t)x[k]) lo[k] = mid; else hi[k] = mid > lo[k] ? mid : lo[k] + 1;
                    more |= hi[k] - lo[k] > 1;
                }
            } while (more);
#pragma unroll
            for (int k = 0; k < AT_ONCE; ++k) m.delta[x[k]] = rowstart[lo[k]] - (eoff[lo[k]] - c0);
        }
        if (threadIdx.x < EdgeMap<TILE>::WORDS) m.starts[threadIdx.x] = ~0ull;
        __syncthreads();
        return off < INT32_MIN ? INT32_MIN : (int32_t)off;
    }
    for (int32_t a = r.first + (int32_t)threadIdx.x; a < r.end;) {
        const int64_t beg = row.beg - c0, end = row.end - c0;
        if (end > beg && end > 0 && beg < len) {
            const int32_t p = beg > 0 ? (int32_t)beg : 0;
            m.delta[p] = row.csr - beg;
            atomicOr(&m.starts[p >> 6], 1ull << (p & 63));
        }
        a += (int32_t)blockDim.x;
        if (a < r.end) row = row_edges(eoff, rowstart, nS, a);
    }
    __syncthreads();
    return off < INT32_MIN ? INT32_MIN : (int32_t)off;
}

// A lane's view of the words: their bits, and the last start at or before the end of each (lane l: word l).
struct EdgeWords {
    uint32_t lo, hi;
    int32_t last;
};
template <int TILE>
__device__ inline EdgeWords edge_words(const EdgeMap<TILE> &m)
{
    const int lane = lane_id();
    const unsigned long long w = lane < EdgeMap<TILE>::WORDS ? m.starts[lane] : 0ull;
    int32_t last = w ? lane * WAVE + 64 - __clzll((long long)w) : 0;   // one past the position; 0: none
    // inclusive maximum over the lanes (zero fill does not change a maximum of counts)
    auto step = [&](uint32_t v) { last = (int32_t)v > last ? (int32_t)v : last; };
    step(dpp_move<0x111, 0xF>((uint32_t)last));
    step(dpp_move<0x112, 0xF>((uint32_t)last));
    step(dpp_move<0x114, 0xF>((uint32_t)last));
    step(dpp_move<0x118, 0xF>((uint32_t)last));
    if (EdgeMap<TILE>::WORDS > 16) {
        step(dpp_move<0x142, 0xA>((uint32_t)last));
        step(dpp_move<0x143, 0xC>((uint32_t)last));
    }
    return EdgeWords{(uint32_t)w, (uint32_t)(w >> 32), last > 0 ? last - 1 : 0};
}
// CSR address of position word * 64 + lane; `word` is the same for the whole wavefront.
template <int TILE>
__device__ inline int64_t edge_address(const EdgeMap<TILE> &m, const EdgeWords &e, int word)
{
    const int lane = lane_id();
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)e.lo, word), hi = (uint32_t)__builtin_amdgcn_readlane((int)e.hi, word);
    const int32_t before = word ? __builtin_amdgcn_readlane(e.last, word - 1) : 0;
    const uint64_t upto = (((uint64_t)hi << 32) | lo) & (~0ull >> (63 - lane));
    const int32_t p = upto ? word * WAVE + 63 - __clzll((long long)upto) : before;
    return m.delta[p] + (word * WAVE + lane);
}

}  // namespace csgs
