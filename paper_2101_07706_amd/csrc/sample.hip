// csgs_draw_nodes, csgs_sampled_adjacency, csgs_sample_layer and csgs_remote_count.
//
// B draws with replacement from the skewed distribution (Section 4.1: the sampling is run B
// times), deduplicated; inclusion probability p_j = 1 - (1 - q_j)^B (Eq. 8); sampled adjacency
// with every kept edge divided by p_j (Eq. 3); number of sampled remote nodes (Eq. 4).
//
// Kernels:
//   draw          one thread per draw: Philox4x32-10 word -> u = mulhi(r, total) -> first cdf
//                 entry above u.  The top levels of the search run on a strided sample of the
//                 CDF staged in LDS, the rest is an 8-ary search on the global array (seven
//                 independent probes per round).  Hits are counted per candidate position with
//                 integer atomics; first hits set a position bitmap.
//   hits          every block takes a range of the position bitmap, counts the bits before it
//                 itself (or, in a long bitmap, takes them from the scan across blocks), lists its own hits in LDS, then one thread per distinct hit: S_next
//                 ascending, mult, p_incl, node -> rank table.
//   adj_mark      flat over the edges of S (same chunking as the weight scan): keep = the target was
//                 sampled.  Leaves every chunk's kept edges in order, their number, and the row
//                 pointers relative to the chunk.  The node -> rank table is never cleared: its
//                 entries carry the tag of the draw that wrote them.
//   adj_place     the kept edges in flat order ARE the CSR of P~ (rows in the order of S, columns
//                 ascending): adds up the counts of the chunks before and puts a chunk's kept edges
//                 and row pointers where they belong
//   adj_once      both in one pass, the prefix by the single-pass scan across blocks: for calls with
//                 few chunks, where a launch costs more than the wait
//   remote_count_k  S_next ascends and the local partition is one id range: two searches by a
//                 whole wavefront place every element (see the kernel)
#include <math.h>
#include "common.hpp"
#include "lookback.hpp"
#include "row_prefix.hpp"

namespace csgs {

// Philox4x32 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC'11): each round multiplies two
// counter words by fixed odd constants, swaps halves around and xors in the key, then the key
// advances by two Weyl increments.
__device__ inline uint64_t philox_word(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0;
        const uint32_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return (uint64_t)c0 | ((uint64_t)c1 << 32);
}

// Blocks of two wavefronts and few samples: the search is bound by the scattered loads of one compute unit, and every sample
// is a line of its own (us for one mini-batch of 8192 draws from 163 K candidates / eight of them / 131 K draws from 650 K: 256
// threads and 2048 samples 10.0 / 16.4 / 26, 128 and 256 7.2 / 15.4 / 24, 64 and 512 8.4 / 16.3 / 26, 1024 and 2048 19 / 24 / 26).
constexpr int DRAW_BLOCK = 128;
constexpr int TOP = 256;   // CDF samples staged in LDS per block

__global__ __launch_bounds__(DRAW_BLOCK) void draw(const uint64_t *__restrict__ cdf,
                                                   const csgs_prob_stats *__restrict__ stats, int64_t cand_cap,
                                                   int32_t B, uint32_t seed_lo, uint32_t seed_hi, uint64_t iter,
                                                   const uint64_t *__restrict__ iter_dev, uint32_t layer,
                                                   uint32_t *__restrict__ hit, uint64_t *cbitmap0, uint64_t *cbitmap1,
                                                   uint64_t *__restrict__ epoch, uint64_t *__restrict__ rank,
                                                   uint64_t *__restrict__ member, int64_t n_nodes, InstStride is)
{
    const InstBlock ib = inst_block(is, true);   // (as many draws for every instance)
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block, n_blk = ib.blocks;
    __shared__ uint64_t top[TOP];
    cdf = inst_ptr(cdf, is.buf); stats = inst_ptr(stats, is.buf);
    hit = inst_ptr(hit, is.ws); cbitmap0 = inst_ptr(cbitmap0, is.ws); cbitmap1 = inst_ptr(cbitmap1, is.ws); epoch = inst_ptr(epoch, is.ws); rank = inst_ptr(rank, is.ws);
    member = inst_ptr(member, is.ws);
    // rank entries and membership words carry the low 32 bits of the call number; when those wrap, stale
    // entries could look current, so both tables are wiped once every 2^32 calls (the compaction kernel that
    // follows writes the new entries)
    if ((call_number(epoch) & 0xFFFFFFFFull) == 0) {
        for (int64_t i = (int64_t)blk * blockDim.x + threadIdx.x; i < n_nodes; i += (int64_t)n_blk * blockDim.x) {
            rank[i] = 0ull;
            if (i < (n_nodes + 31) / 32) member[i] = 0ull;
        }
    }
    if (iter_dev) iter = *iter_dev;
    iter += ib.k;   // consecutive instances are consecutive iterations
    const uint32_t iter_lo = (uint32_t)iter, iter_hi = (uint32_t)(iter >> 32);
    int64_t n = stats->n_cand;
    if (n > cand_cap) n = cand_cap;
    const uint64_t turn = epoch[EPOCH_BITMAP_NEXT] & 1ull;
    uint64_t *__restrict__ cbitmap = turn ? cbitmap1 : cbitmap0;
    if (blk == 0 && threadIdx.x == 0) {   // (nobody reads these words in this kernel)
        epoch[EPOCH_DRAW] = call_number(epoch);
        epoch[EPOCH_BITMAP_CUR] = turn;
        epoch[EPOCH_BITMAP_USED + turn] = (uint64_t)(n > 0 ? (n + 63) / 64 : 0);
    }
    if (n <= 0) return;
    const uint64_t total = stats->total;   // = cdf[n - 1], without waiting for a second dependent load
    if (total == 0) return;
    // top[i] = cdf[(i + 1) * stride - 1] for the i with that index inside the array
    const int64_t stride = (n + TOP - 1) / TOP;
    const int64_t n_top = n / stride;  // number of complete strides
    for (int64_t i = threadIdx.x; i < n_top; i += blockDim.x) top[i] = cdf[(i + 1) * stride - 1];
    __syncthreads();
    const int64_t t = (int64_t)blk * blockDim.x + threadIdx.x;
    if (t >= B) return;
    const uint64_t r = philox_word((uint32_t)t, layer, iter_lo, iter_hi, seed_lo, seed_hi);
    const uint64_t u = __umul64hi(r, total);
    // first sample above u: the answer lies in stride block a
    int64_t a = 0, b = n_top;
    while (a < b) {
        const int64_t m = (a + b) >> 1;
        if (top[m] > u) b = m; else a = m + 1;
    }
    int64_t lo = a * stride;
    int64_t hi = (a < n_top) ? (a + 1) * stride - 1 : n - 1;  // cdf[hi] > u is known; the answer is in [lo, hi]
    // 8-ary search on the global array: 7 independent probes per round instead of one
    while (hi - lo >= 8) {
        const int64_t len = hi - lo;  // candidates lo .. hi, hi already known to be above u
        uint64_t pv[7];
#pragma unroll
        for (int i = 0; i < 7; ++i) pv[i] = cdf[lo + (len * (i + 1)) / 8];
        int below = 0;                // pivots that are <= u (they ascend, so these are the first ones)
#pragma unroll
        for (int i = 0; i < 7; ++i) below += pv[i] <= u ? 1 : 0;
        const int64_t new_lo = below ? lo + (len * below) / 8 + 1 : lo;
        const int64_t new_hi = below < 7 ? lo + (len * (below + 1)) / 8 : hi;
        lo = new_lo;
        hi = new_hi;
    }
    {
        // at most 8 entries left: fetch them together, take the first above u
        uint64_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (lo + i < hi) ? cdf[lo + i] : ~0ull;
        int skip = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) skip += v[i] <= u ? 1 : 0;
        lo += skip;  // entries ascend; cdf[hi] > u bounds the result by hi
        if (lo > hi) lo = hi;
    }
    // both updates are fire-and-forget (no returned value to wait for); setting an already set bit is harmless
    (void)__hip_atomic_fetch_add(&hit[lo], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    (void)__hip_atomic_fetch_or((unsigned long long *)&cbitmap[lo >> 6], 1ull << (lo & 63), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
}

// The membership words: word id / 32 holds (tag << 32) | one bit per id, set when the id is in S_next of the draw
// with that tag; the adjacency pass looks an edge's column up here (612 KB for 2.4 M nodes: it stays in the L2s)
// and goes to the 8-byte-per-node rank table only for the one column in twenty that is a member.
// Merging bits into a word that other wavefronts may write as well: a word of an older draw counts as empty.  Two
// updates nobody waits for: a 64-bit maximum with (tag << 32) replaces an older draw's word by the empty word of this
// draw and leaves a current one alone (tags ascend from draw to draw; the table is wiped when they wrap), then the
// bits are or-ed in.  Updates of one address by one lane take effect in program order.
__device__ inline void member_merge(uint64_t *word, uint32_t bits, uint32_t tag32)
{
    unsigned long long *p = reinterpret_cast<unsigned long long *>(word);
    (void)__hip_atomic_fetch_max(p, (unsigned long long)tag32 << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    (void)__hip_atomic_fetch_or(p, (unsigned long long)bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every lane of a wavefront calls this with the id of its hit (-1: none).  The hits of a wavefront are consecutive
// entries of the ascending list, so the ids that share a word sit in neighbouring lanes: their bits are put
// together by lane exchanges and the first lane of the run stores the word.  All ids of a word that lies strictly
// inside the wavefront's hits are in this wavefront, so that store is a plain one; a run next to a lane without a
// hit, or at either end of the wavefront, may go on in another wavefront and is merged atomically.
__device__ inline void mark_members(uint64_t *__restrict__ member, int32_t id, uint32_t tag32)
{
    const int lane = lane_id();
    const int32_t w = id >= 0 ? id >> 5 : -1;
    uint32_t bits = id >= 0 ? 1u << (id & 31) : 0u;
    const int32_t wp = __shfl_up(w, 1, WAVE), wn = __shfl_down(w, 1, WAVE);
    const bool head = w >= 0 && (lane == 0 || wp != w);
    uint32_t open = (w >= 0 && (lane == WAVE - 1 || wn < 0)) ? 1u : 0u;   // matters in the run's last lane: nothing valid follows it here
#pragma unroll
    for (int d = 1; d <= 16; d <<= 1) {   // a run has at most 32 lanes
        const uint32_t ob = __shfl_down(bits, d, WAVE), oo = __shfl_down(open, d, WAVE);
        const int32_t w2 = __shfl_down(w, d, WAVE);
        if (lane + d < WAVE && w2 == w) { bits |= ob; open |= oo; }
    }
    if (head) {
        if (open || lane == 0 || wp < 0) member_merge(&member[w], bits, tag32);
        else member[w] = ((uint64_t)tag32 << 32) | bits;
    }
}

// The distinct drawn positions in order.  Every block takes `wpb` consecutive words of the position bitmap and counts
// the bits of all words before them itself: the bitmap of n_c positions is n_c / 8 bytes (20 KB for 163 K candidates),
// which a block reads from the L2s in one or two load latencies, where the prefix by waiting for other blocks took
// three.  Nobody waits, so there may be as many blocks as the hits can use: bound by the dependent loads of a hit (bit,
// counter, CDF, id), then by the double-precision logarithm and exponential, which more blocks share.  One mini-batch
// of 8192 draws from 163 K candidates: 16 -> 6 us; 131072 from 650 K: 73 -> 11 us (blocks of 16384 positions with a
// prefix across blocks before).
// A long bitmap is too much for every block to read: beyond HIT_COUNT_WORDS the blocks count their own words and take the
// prefix from the scan across blocks (a block waits for lower ones only, which were dispatched before it).  us, reading all /
// scan, 8192 draws: 1.8 M candidates 10.2 / 11.4, 2.4 M 12.3 / 13.9, 16 M 50 / 26, 256 M 572 / 109.
__global__ __launch_bounds__(256) void hits(const int32_t *__restrict__ cand_id, const uint64_t *__restrict__ cdf,
                                            const csgs_prob_stats *__restrict__ stats, int64_t cand_cap, int64_t n_nodes,
                                            int32_t B, uint64_t *__restrict__ epoch, uint32_t *__restrict__ hit,
                                            uint64_t *cbitmap0, uint64_t *cbitmap1, uint64_t *__restrict__ rank,
                                            uint64_t *__restrict__ member, int32_t *__restrict__ S_next,
                                            int32_t *__restrict__ mult, float *__restrict__ p_incl,
                                            double *__restrict__ pdbl, int32_t *__restrict__ n_next,
                                            uint64_t *__restrict__ ts_mem, int32_t *__restrict__ status, InstStride is)
{
    const InstBlock ib = inst_block(is, epoch[EPOCH_EVEN] != 0);
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block, n_blk = ib.blocks;
    constexpr int SUB = 64;   // words listed at a time: four threads of 16 bits each per word
    __shared__ uint16_t s_list[SUB * 64];   // drawn positions of those words, ascending
    __shared__ uint32_t s_cnt[4], s_before[4];
    __shared__ unsigned long long s_lb[1];
    member = inst_ptr(member, is.ws);
    cand_id = inst_ptr(cand_id, is.buf); cdf = inst_ptr(cdf, is.buf); stats = inst_ptr(stats, is.buf);
    S_next = inst_ptr(S_next, is.buf); mult = inst_ptr(mult, is.buf); p_incl = inst_ptr(p_incl, is.buf);
    n_next = inst_ptr(n_next, is.buf);
    epoch = inst_ptr(epoch, is.ws); hit = inst_ptr(hit, is.ws); cbitmap0 = inst_ptr(cbitmap0, is.ws);
    cbitmap1 = inst_ptr(cbitmap1, is.ws); rank = inst_ptr(rank, is.ws); pdbl = inst_ptr(pdbl, is.ws);
    ts_mem = inst_ptr(ts_mem, is.ws); status = inst_ptr(status, is.buf);
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const unsigned long long call = epoch[EPOCH_DRAW];   // left by the draw
    const uint64_t turn = epoch[EPOCH_BITMAP_CUR];
    const uint64_t *__restrict__ bits = turn ? cbitmap1 : cbitmap0;
    uint64_t *__restrict__ old_bits = turn ? cbitmap0 : cbitmap1;
    const int64_t old_words = (int64_t)epoch[EPOCH_BITMAP_USED + (turn ^ 1ull)];
    int64_t n = stats->n_cand;
    if (n > cand_cap) n = cand_cap;
    if (n < 0) n = 0;
    const double total = (double)stats->total;   // = cdf[n - 1]
    const int64_t n_words = (n + 63) / 64;
    if (blk == 0 && tid == 0) {   // last kernel of the draw (nobody reads these words in this kernel)
        epoch[EPOCH_CALLS] = call;
        epoch[EPOCH_BITMAP_NEXT] = turn ^ 1ull;
        if (n_words == 0) *n_next = 0;
    }
    for (int64_t i = (int64_t)blk * 256 + tid; i < old_words; i += (int64_t)n_blk * 256) old_bits[i] = 0ull;
    int64_t wpb = ((n_words + n_blk - 1) / n_blk + 1) / 2 * 2;   // even
    if (wpb < HIT_MIN_WORDS) wpb = HIT_MIN_WORDS;
    const int64_t w0 = (int64_t)blk * wpb, w1 = w0 + wpb < n_words ? w0 + wpb : n_words;
    if (w0 >= n_words) return;
    const uint64_t rank_tag = (call & 0xFFFFFFFFull) << 32;
    uint64_t word = w0 + (tid >> 2) < w1 ? bits[w0 + (tid >> 2)] : 0ull;
    uint32_t before = 0;   // bits set before w0 (then before the words at hand)
    const bool chained = n_words > HIT_COUNT_WORDS;
    {
        // pairs of words (w0 is even; behind an odd last word lies a zero), eight loads per thread on their way at a time
        const ulonglong2 *__restrict__ pairs = reinterpret_cast<const ulonglong2 *>(bits);
        const int64_t end = ((chained ? w1 : w0) + 1) / 2;
        uint32_t c = 0;
        for (int64_t i = (chained ? w0 / 2 : 0) + tid; i < end; i += 8 * 256) {
            ulonglong2 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = pairs[i + k * 256 < end ? i + k * 256 : i];
#pragma unroll
            for (int k = 0; k < 8; ++k) c += i + k * 256 < end ? (uint32_t)(__popcll(v[k].x) + __popcll(v[k].y)) : 0u;
        }
        c = wave_sum(c);
        if (lane == 0) s_before[wave] = c;
    }
    if (chained) {
        const TileState<1> ts(ts_mem, HIT_GRID, wait_limit(epoch));
        const unsigned long long tag = call_tag(call, SLOT_HITS);
        __syncthreads();
        // (a count and one in the bits above it, so that no sum of these is ever taken for a tag)
        const unsigned long long local[1] = {(1ull << 52) + s_before[0] + s_before[1] + s_before[2] + s_before[3]};
        unsigned long long excl[1];
        lookback_publish<1>(ts, tag, blk, local);
        lookback_resolve<1>(ts, tag, blk, (n_words + wpb - 1) / wpb, local, excl, s_lb, status);
        before = (uint32_t)excl[0];   // (positions: below 2^31)
    }
    for (int64_t ws = w0; ws < w1; ws += SUB) {
        if (ws > w0) word = ws + (tid >> 2) < w1 ? bits[ws + (tid >> 2)] : 0ull;
        uint32_t mine = (uint32_t)(word >> (16 * (tid & 3))) & 0xFFFFu;
        const uint32_t cnt = (uint32_t)__popc(mine);
        const uint32_t incl = wave_inclusive_scan(cnt);
        if (lane == WAVE - 1) s_cnt[wave] = incl;
        __syncthreads();
        if (ws == w0 && !chained) before = s_before[0] + s_before[1] + s_before[2] + s_before[3];
        uint32_t at = incl - cnt, n_hits = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t c = s_cnt[k];
            if (k < wave) at += c;
            n_hits += c;
        }
        while (mine) {
            const int bit = __ffs((int)mine) - 1;
            mine &= mine - 1;
            s_list[at++] = (uint16_t)(tid * 16 + bit);
        }
        __syncthreads();
        for (uint32_t i0 = 0; i0 < n_hits; i0 += 256) {   // every lane goes round together (mark_members)
            const uint32_t i = i0 + (uint32_t)tid;
            int32_t member_id = -1;
            if (i < n_hits) {
                const int64_t kpos = ws * 64 + s_list[i];
                const uint32_t m = hit[kpos];
                const uint64_t hi = cdf[kpos], lo = cdf[kpos > 0 ? kpos - 1 : 0];
                const int32_t id = cand_id[kpos];
                const double qk = (double)(kpos > 0 ? hi - lo : hi) / total;
                const double pk = (qk >= 1.0) ? 1.0 : -expm1((double)B * log1p(-qk));
                hit[kpos] = 0u;   // back to the clean state
                const uint64_t pos = (uint64_t)before + i;
                if (pos < (uint64_t)B) {  // at most B distinct hits exist; the guard keeps stores in bounds regardless
                    S_next[pos] = id;
                    mult[pos] = (int32_t)m;
                    p_incl[pos] = (float)pk;
                    pdbl[pos] = pk;
                    if (id >= 0 && id < n_nodes) {
                        rank[id] = rank_tag | (pos + 1);
                        member_id = id;
                    }
                }
            }
            mark_members(member, member_id, (uint32_t)(rank_tag >> 32));
        }
        before += n_hits;
        __syncthreads();   // the list is written again
    }
    if (w1 == n_words && tid == 0) *n_next = (int32_t)(before < (uint32_t)B ? before : (uint32_t)B);
}

// S_next ascends and the local partition is one id range, so the sampled remote nodes are the
// entries before the first id >= lo and from the first id >= hi on: two searches give every
// element its place, no scan needed.
// Blocks of 256 threads that cover a budget of B and, a partition per wavefront, the P partitions in one sweep; more are
// strided over.  (us of the one-pass adjacency, blocks by B alone / this: 200 draws, 1024 partitions 206 / 10, 256 partitions
// 53 / 10.)
static int remote_blocks(int64_t B, int64_t P)
{
    const int64_t n = (B + 255) / 256 > (P + 3) / 4 ? (B + 255) / 256 : (P + 3) / 4;
    return (int)(n < 1 ? 1 : (n < 256 ? n : 256));
}

struct RemoteArgs {
    const int32_t *S_next, *n_next;
    int32_t lo, hi;
    const int32_t *part_bounds;
    int32_t P;
    int64_t *remote_total, *per_part;
    int32_t *src_row, *remote_ids;
    int32_t blocks;   // blocks of 256 threads that do this work (as leading blocks of another kernel: 0 = none)
};

// `block` of `n_blocks` blocks of 256 threads
__device__ inline void remote_count_body(const RemoteArgs &r_, int32_t block, int32_t n_blocks)
{
    const int32_t *__restrict__ S_next = r_.S_next;
    const int32_t lo = r_.lo, hi = r_.hi, P = r_.P;
    const int32_t *__restrict__ part_bounds = r_.part_bounds;
    int64_t *__restrict__ remote_total = r_.remote_total, *__restrict__ per_part = r_.per_part;
    int32_t *__restrict__ src_row = r_.src_row, *__restrict__ remote_ids = r_.remote_ids;
    int32_t n = *r_.n_next;
    if (n < 0) n = 0;
    // ids below the local range end at a, the first id above it is at b
    int32_t ab[2];
    const int32_t bounds[2] = {lo, hi};
    wave_lower_bounds<2>(S_next, n, bounds, ab);
    const int32_t a = ab[0], b = ab[1];
    const int32_t n_local = b - a;
    const int32_t tid = (int32_t)(block * blockDim.x + threadIdx.x);
    const int32_t stride = (int32_t)(n_blocks * blockDim.x);
    if (tid == 0) *remote_total = (int64_t)(n - n_local);
    if (src_row || remote_ids) {
        for (int32_t k = tid; k < n; k += stride) {
            const int32_t j = S_next[k];
            if (k >= a && k < b) {
                if (src_row) src_row[k] = j - lo;
            } else {
                const int32_t r = k < a ? k : k - n_local;
                if (src_row) src_row[k] = -1 - r;
                if (remote_ids && r >= 0 && r < n) remote_ids[r] = j;   // (r leaves [0, n) only if S_next does not ascend)
            }
        }
    }
    // partition p holds the ids between two lower bounds; one wavefront per partition
    if (per_part) {
        const int32_t wave = tid >> 6, n_waves = stride >> 6;
        for (int32_t p = wave; p < P; p += n_waves) {
            const int32_t ends[2] = {part_bounds[p], part_bounds[p + 1]};
            int32_t c[2];
            wave_lower_bounds<2>(S_next, n, ends, c);
            if (lane_id() == 0) per_part[p] = (int64_t)(c[1] > c[0] ? c[1] - c[0] : 0);
        }
    }
}

__global__ __launch_bounds__(256) void remote_count_k(RemoteArgs r) { remote_count_body(r, (int32_t)blockIdx.x, (int32_t)gridDim.x); }

// Work of the marking pass's second group of spare blocks: the row offsets of the node set just
// sampled, for a following csgs_build_probs on those rows (one tile of rows per block).
struct NextRows {
    const int64_t *rowptr;
    int64_t n_nodes;
    const int32_t *S_next, *n_next;
    int32_t bound;        // capacity of S_next (the B of the draw)
    uint64_t *ts_mem;
    int64_t ts_tiles;
    int64_t *eoff, *rowstart, *meta;
    int2 *bound_note;
    int64_t edge_cap;
    int32_t blocks;       // 0 = none
};

// One chunk of edges: which of them are kept.  Called by all threads; wavefront w owns positions [w * 256, w * 256 + 256),
// four 64-edge words.  Out: per lane and word the kept edge's rank (position in S_next + 1; 0 = not kept) and CSR
// position; in LDS the keep bits of every word (mask) and the kept edges before it (pre).
struct AdjChunk {
    EdgeMap<EDGE_TILE> map;
    uint64_t mask[EDGE_TILE / 64];
    int32_t pre[EDGE_TILE / 64 + 1];
};
struct AdjGraph {
    const int32_t *colidx;
    const float *val;
    int64_t n_nodes, nnz;
    const int64_t *eoff, *rowstart;
    const uint64_t *rank, *member;
    const double *pdbl;
};
// Returns what map_edges() does.
__device__ inline int32_t adj_chunk(AdjChunk &s, const AdjGraph &g, int32_t nS, int64_t c0, int64_t c1, uint64_t rank_tag, ChunkRows &rows,
                                    int32_t (&rk)[4], int64_t (&ea)[4])
{
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const int32_t len = (int32_t)(c1 - c0);
    const int32_t starts = map_edges(s.map, g.eoff, g.rowstart, nS, c0, len, rows, first_rows(g.eoff, g.rowstart, nS, rows));
    const EdgeWords words = edge_words(s.map);
    // A lane's four edges go through each step together, and no load sits under a condition (an edge that does
    // not exist reads entry 0 and is dropped): the four columns travel at the same time, then the four table
    // lookups, instead of eight trips one after the other.
    bool live[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int32_t x = wave * 256 + k * 64 + lane;
        const int64_t a = edge_address(s.map, words, __builtin_amdgcn_readfirstlane(wave * 4 + k));
        live[k] = x < len && a >= 0 && a < g.nnz;   // (an address outside the graph can only follow a failed wait)
        ea[k] = live[k] ? a : 0;
    }
    int32_t ck[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) ck[k] = g.colidx[ea[k]];
    // the membership word of every column first (a small table that stays in the L2s), then the rank entry, which
    // only a member's lane reads from its own place (the others read entry 0)
    uint64_t mw[4], re[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        live[k] = live[k] && ck[k] >= 0 && ck[k] < g.n_nodes;
        mw[k] = g.member[live[k] ? ck[k] >> 5 : 0];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        live[k] = live[k] && (mw[k] & 0xFFFFFFFF00000000ull) == rank_tag && ((mw[k] >> (ck[k] & 31)) & 1ull);
        re[k] = g.rank[live[k] ? ck[k] : 0];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        rk[k] = (live[k] && (re[k] & 0xFFFFFFFF00000000ull) == rank_tag) ? (int32_t)(re[k] & 0xFFFFFFFFull) : 0;
        const uint64_t m = __ballot(rk[k] > 0);
        if (lane == 0) s.mask[wave * 4 + k] = m;
    }
    __syncthreads();
    if (wave == 0) {
        const int32_t c = lane < EDGE_TILE / 64 ? __popcll(s.mask[lane]) : 0;
        const int32_t incl = wave_inclusive_scan(c);
        if (lane <= EDGE_TILE / 64) s.pre[lane] = incl - c;
    }
    __syncthreads();
    return starts;
}
// Kept edges of the chunk before position `off` of it (0 <= off < its length)
__device__ inline int32_t kept_before(const AdjChunk &s, int32_t off)
{
    return s.pre[off >> 6] + __popcll(s.mask[off >> 6] & ((1ull << (off & 63)) - 1ull));
}
// Value and place inside the chunk of a lane's kept edges (unconditional loads again)
__device__ inline void adj_values(const AdjChunk &s, const AdjGraph &g, const int32_t (&rk)[4], const int64_t (&ea)[4], float (&pv)[4],
                                  int32_t (&at)[4])
{
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    float vv[4];
    double pp[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        vv[k] = g.val[ea[k]];
        pp[k] = g.pdbl[rk[k] > 0 ? rk[k] - 1 : 0];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int32_t word = wave * 4 + k;
        pv[k] = rk[k] > 0 ? (float)((double)vv[k] / pp[k]) : 0.f;
        at[k] = s.pre[word] + __popcll(s.mask[word] & ((1ull << lane) - 1ull));
    }
}

// The leading blocks of an adjacency kernel do two other things that need only the new node set, complete since the
// previous kernel, so that a layer step is that many launches shorter.  Returns true for such a block.
__device__ inline bool adj_leading_blocks(RemoteArgs &rem, NextRows &nxt, const uint64_t *__restrict__ epoch, int32_t *__restrict__ status,
                                          const InstStride &is, uint32_t blk)
{
    // The first rem.blocks split the node set into local and remote (what csgs_remote_count does); they wait for nobody
    // and nobody waits for them.
    if ((int32_t)blk < rem.blocks) {
        rem.S_next = inst_ptr(rem.S_next, is.buf); rem.n_next = inst_ptr(rem.n_next, is.buf);
        rem.remote_total = inst_ptr(rem.remote_total, is.buf); rem.per_part = inst_ptr(rem.per_part, is.buf);
        rem.src_row = inst_ptr(rem.src_row, is.buf); rem.remote_ids = inst_ptr(rem.remote_ids, is.buf);
        remote_count_body(rem, (int32_t)blk, rem.blocks);
        return true;
    }
    // The next nxt.blocks lay out the rows of the new node set.  They wait only for each other (lower tiles, dispatched
    // before them); their flags are tagged with the draw's call number, so the counter that a call's last kernel
    // advances does not matter.
    if ((int32_t)blk < rem.blocks + nxt.blocks) {
        nxt.S_next = inst_ptr(nxt.S_next, is.buf); nxt.n_next = inst_ptr(nxt.n_next, is.buf);
        nxt.ts_mem = inst_ptr(nxt.ts_mem, is.ws); nxt.eoff = inst_ptr(nxt.eoff, is.ws);
        nxt.rowstart = inst_ptr(nxt.rowstart, is.ws); nxt.meta = inst_ptr(nxt.meta, is.ws);
        nxt.bound_note = inst_ptr(nxt.bound_note, is.ws);
        const int32_t n = resolve_count(nxt.bound, nxt.n_next);
        const int64_t t = (int64_t)blk - rem.blocks, n_tiles = row_tiles(n);
        if (t < n_tiles) {
            const TileState<1> rts(nxt.ts_mem, nxt.ts_tiles, wait_limit(epoch));
            row_prefix_tile(nxt.rowptr, nxt.n_nodes, nxt.S_next, n, t, n_tiles, rts, call_tag(epoch[EPOCH_DRAW], SLOT_ROWS_NEXT),
                            nxt.eoff, nxt.rowstart, nxt.meta, nxt.edge_cap, nxt.bound_note, nxt.edge_cap / EDGE_TILE, status);
        }
        return true;
    }
    return false;
}

// Two passes over the edges' chunks, neither of which waits: the first does everything that costs lookups, with as many
// blocks as the device holds; the second only adds up 4 bytes per chunk and copies what was kept.  Against the one pass
// below, whose 512 resident blocks wait for each other's counts once per round (us per layer): 6.6 M edges 84 / 139, 4.1 M
// 54 / 90, eight mini-batches of 380 K 35 / 41, 957 K 15 / 22; level at 413 K (16 / 15); beyond the 8 Mi edges whose kept ones
// the first pass can leave, where the second looks up the rest again: 16.7 M 300 / 340, 33 M 645 / 720, 125 M 2310 / 3500.  The first
// pass is bound by its random lookups in the membership words (100 G edges/s).
// Most chunks (of all instances of a launch, as expected from the mean degree with a quarter to spare) for the one pass: with one instance while
// every chunk has a block of its own.  (us of csgs_build_probs and csgs_sample_layer, 1 K to 65 K draws, two passes / one.  200 K nodes: 2 K edges 50 to
// 100 / 48 to 90, 259 K 58 to 99 / 57 to 93, 408 K 63 to 104 / 61 to 97; 2.4 M nodes: 259 K 64 to 77 / 63 to 75, 408 K 66 to 79 / 64 to 76; beyond a chunk per block
// level or dearer.  Rows of hubs that hold many times what the mean expects are dearer in one pass, whose blocks a compute unit holds
// fewer of: 1.4 M edges where 0.4 M are expected 136 / 148, 4.4 M 284 / 324.)  With several instances the line is where it was measured for them.
constexpr int ADJ_ONCE_MAX = 560, ADJ_ONCE_MAX_EACH = 256;
constexpr int ADJ_MARK_GRID = 2048;    // eight blocks per compute unit, by threads
constexpr int ADJ_PLACE_GRID = 512;
constexpr int ADJ_PLACE_MIN = 4;       // chunks a block of the placing pass takes at least: one per wavefront

__global__ __launch_bounds__(256) void adj_mark(AdjGraph g, const int64_t *__restrict__ meta, const uint64_t *__restrict__ epoch,
                                                int64_t chunk_cap, const int2 *__restrict__ bound_note, uint32_t *__restrict__ chunk_cnt,
                                                uint64_t *__restrict__ kept, int64_t kept_chunks, int32_t *__restrict__ adj_rowptr,
                                                int32_t *__restrict__ status, RemoteArgs rem, NextRows nxt, InstStride is)
{
    const InstBlock ib = inst_block(is, epoch[EPOCH_EVEN] != 0);
    is = at_instance(is, ib.k);
    const uint32_t blk = ib.block, n_blk = ib.blocks;
    epoch = inst_ptr(epoch, is.ws); status = inst_ptr(status, is.buf);
    if (adj_leading_blocks(rem, nxt, epoch, status, is, blk)) return;
    meta = inst_ptr(meta, is.ws); g.eoff = inst_ptr(g.eoff, is.ws); g.rowstart = inst_ptr(g.rowstart, is.ws);
    g.rank = inst_ptr(g.rank, is.ws); g.member = inst_ptr(g.member, is.ws); g.pdbl = inst_ptr(g.pdbl, is.ws);
    bound_note = inst_ptr(bound_note, is.ws); chunk_cnt = inst_ptr(chunk_cnt, is.ws); kept = inst_ptr(kept, is.ws);
    adj_rowptr = inst_ptr(adj_rowptr, is.buf);
    const int64_t bid = (int64_t)blk - rem.blocks - nxt.blocks;
    const int64_t n_bids = (int64_t)n_blk - rem.blocks - nxt.blocks;
    ChunkRows rows = chunk_rows(bound_note, bid, bid + 1);   // (the grid stays within the notes; on its way beside the counts)
    __shared__ AdjChunk s;
    const uint64_t rank_tag = (epoch[EPOCH_DRAW] & 0xFFFFFFFFull) << 32;
    const int32_t nS = (int32_t)meta[META_ROWS];
    const int64_t E = meta[META_EDGES];
    const int64_t n_chunks = (E + EDGE_TILE - 1) / EDGE_TILE;
    if (n_chunks > chunk_cap) return;   // (adj_place reports it)
    for (int64_t t = bid; t < n_chunks; t += n_bids) {
        const int64_t c0 = t * EDGE_TILE;
        const int64_t c1 = (c0 + EDGE_TILE < E) ? c0 + EDGE_TILE : E;
        int32_t rk[4], at[4];
        int64_t ea[4];
        float pv[4];
        if (t != bid) rows = chunk_rows(bound_note, t, t + 1);
        int32_t off = adj_chunk(s, g, nS, c0, c1, rank_tag, rows, rk, ea);
        adj_values(s, g, rk, ea, pv, at);
        if (threadIdx.x == 0) chunk_cnt[t] = (uint32_t)s.pre[EDGE_TILE / 64] | (off == 0 ? 0x80000000u : 0u);
        // row pointers of the rows that start inside this chunk (the last one's: or behind it): kept edges of the chunk before the row start
        const int32_t len = (int32_t)(c1 - c0);
        const bool last = t == n_chunks - 1;
        for (int32_t a = rows.first + (int32_t)threadIdx.x; a < rows.end;) {
            if (off >= 0 && (off < len || last)) adj_rowptr[a] = off < len ? kept_before(s, off) : s.pre[EDGE_TILE / 64];
            a += (int32_t)blockDim.x;
            if (a < rows.end) off = (int32_t)(g.eoff[a] - c0);   // (a row behind the first one starts inside the chunk or at its end)
        }
        if (t < kept_chunks) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (rk[k] > 0) kept[t * EDGE_TILE + at[k]] = (uint64_t)(uint32_t)(rk[k] - 1) | ((uint64_t)__float_as_uint(pv[k]) << 32);
        }
    }
}

__global__ __launch_bounds__(256) void adj_place(AdjGraph g, const int64_t *__restrict__ meta, uint64_t *__restrict__ epoch,
                                                 int64_t chunk_cap, const int2 *__restrict__ bound_note, const uint32_t *__restrict__ chunk_cnt,
                                                 const uint64_t *__restrict__ kept, int64_t kept_chunks, int32_t *__restrict__ adj_rowptr,
                                                 int32_t *__restrict__ adj_col, float *__restrict__ adj_val, int64_t adj_cap,
                                                 int64_t *__restrict__ adj_nnz, int32_t *__restrict__ status, InstStride is)
{
    is = at_instance(is);
    const uint32_t blk = blockIdx.x, n_blk = gridDim.x;
    __shared__ uint32_t s_scan[17];
    __shared__ uint32_t s_cnt[256], s_base[256];
    __shared__ ChunkRows s_rows[256];
    __shared__ uint64_t s_sum[4];
    __shared__ AdjChunk s;   // only for chunks whose kept edges were not left (more than kept_chunks)
    status = inst_ptr(status, is.buf); epoch = inst_ptr(epoch, is.ws);
    meta = inst_ptr(meta, is.ws); g.eoff = inst_ptr(g.eoff, is.ws); g.rowstart = inst_ptr(g.rowstart, is.ws);
    g.rank = inst_ptr(g.rank, is.ws); g.member = inst_ptr(g.member, is.ws); g.pdbl = inst_ptr(g.pdbl, is.ws);
    bound_note = inst_ptr(bound_note, is.ws); chunk_cnt = inst_ptr(chunk_cnt, is.ws); kept = inst_ptr(kept, is.ws);
    adj_rowptr = inst_ptr(adj_rowptr, is.buf); adj_col = inst_ptr(adj_col, is.buf); adj_val = inst_ptr(adj_val, is.buf);
    adj_nnz = inst_ptr(adj_nnz, is.buf);
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int32_t nS = (int32_t)meta[META_ROWS];
    // Row pointers never exceed what adj_col / adj_val can hold: when the kept edges overflow the
    // capacity (status bit), later kernels that walk the rows still stay inside the arrays.
    const int64_t ptr_max = adj_cap < 0x7FFFFFFFll ? adj_cap : 0x7FFFFFFFll;
    int64_t E = meta[META_EDGES];
    int64_t n_chunks = (E + EDGE_TILE - 1) / EDGE_TILE;
    const bool overflow = n_chunks > chunk_cap;   // the workspace cannot describe this many chunks: report, emit nothing
    if (overflow) { E = 0; n_chunks = 0; }
    if (blk == 0 && tid == 0) {
        epoch[EPOCH_CALLS] += 1ull;   // last kernel of the call; no block of this kernel or of the marking pass reads the counter
        if (overflow) atomicOr(status, CSGS_ST_EDGE_OVERFLOW);
        if (n_chunks == 0) *adj_nnz = 0;
    }
    if (n_chunks == 0) {
        if (blk == 0)
            for (int32_t a = tid; a <= nS; a += 256) adj_rowptr[a] = 0;
        return;
    }
    int64_t per = (n_chunks + n_blk - 1) / n_blk;
    if (per < ADJ_PLACE_MIN) per = ADJ_PLACE_MIN;
    const int64_t t0 = (int64_t)blk * per, t1 = t0 + per < n_chunks ? t0 + per : n_chunks;
    if (t0 >= n_chunks) return;
    constexpr uint32_t CNT = 0x7FFFFFFFu;
    uint64_t base = 0;   // kept edges before chunk t0 (then before the chunks at hand)
    {
        uint64_t c = 0;
        int64_t i = tid;
        for (; i + 3 * 256 < t0; i += 4 * 256)
            c += (uint64_t)(chunk_cnt[i] & CNT) + (chunk_cnt[i + 256] & CNT) + (chunk_cnt[i + 512] & CNT) + (chunk_cnt[i + 768] & CNT);
        for (; i < t0; i += 256) c += chunk_cnt[i] & CNT;
        c = wave_sum(c);
        if (lane == 0) s_sum[wave] = c;
    }
    for (int64_t ts = t0; ts < t1; ts += 256) {
        const int m = (int)(t1 - ts < 256 ? t1 - ts : 256);
        const uint32_t raw = tid < m ? chunk_cnt[ts + tid] : 0u;
        if (tid < m) s_rows[tid] = chunk_rows(bound_note, ts + tid, ts + tid + 1);
        uint32_t sum;
        const uint32_t ex = block_exclusive_scan<uint32_t>(raw & CNT, s_scan, &sum);   // (starts with a barrier: the arrays below are free)
        s_cnt[tid] = raw;
        s_base[tid] = ex;
        if (ts == t0) base = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        __syncthreads();
        for (int k = wave; k < m; k += 4) {   // one wavefront per chunk
            const int64_t t = ts + k;
            const uint32_t cnt = s_cnt[k] & CNT;
            const int64_t b = (int64_t)(base + s_base[k]);
            int64_t a = s_rows[k].first, a_end = s_rows[k].end;   // (stay inside the row pointers whatever a broken prefix left)
            if (!(s_cnt[k] >> 31)) ++a;                        // the chunk's first row began in an earlier chunk
            if (a < 0) a = 0;
            if (a_end > nS) a_end = nS;
            for (int64_t r = a + lane; r < a_end; r += WAVE) {
                const int64_t v = b + adj_rowptr[r];
                adj_rowptr[r] = (int32_t)(v < ptr_max ? v : ptr_max);
            }
            if (t < kept_chunks)
                for (uint32_t i = lane; i < cnt; i += WAVE) {
                    const uint64_t e = kept[t * EDGE_TILE + i];
                    if (b + i < adj_cap) {
                        adj_col[b + i] = (int32_t)(uint32_t)e;
                        adj_val[b + i] = __uint_as_float((uint32_t)(e >> 32));
                    }
                }
        }
        for (int64_t t = ts > kept_chunks ? ts : kept_chunks; t < ts + m; ++t) {   // not left by the marking pass: look them up again
            const int64_t c0 = t * EDGE_TILE, c1 = (c0 + EDGE_TILE < E) ? c0 + EDGE_TILE : E;
            int32_t rk[4], at[4];
            int64_t ea[4];
            float pv[4];
            ChunkRows rows = chunk_rows(bound_note, t, t + 1);
            adj_chunk(s, g, nS, c0, c1, (epoch[EPOCH_DRAW] & 0xFFFFFFFFull) << 32, rows, rk, ea);
            adj_values(s, g, rk, ea, pv, at);
            const int64_t b = (int64_t)(base + s_base[t - ts]);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (rk[k] > 0 && b + at[k] < adj_cap) {
                    adj_col[b + at[k]] = rk[k] - 1;
                    adj_val[b + at[k]] = pv[k];
                }
        }
        base += sum;
        __syncthreads();
    }
    if (t1 == n_chunks) {
        // rows behind the last one with edges, and the end pointer
        const int64_t total = (int64_t)base;
        const int32_t clamp = (int32_t)(total < ptr_max ? total : ptr_max);
        const int32_t end = chunk_rows(bound_note, n_chunks - 1, n_chunks).end;
        for (int64_t a = (end < 0 ? 0 : end) + (int64_t)tid; a <= nS; a += 256) adj_rowptr[a] = clamp;
        if (tid == 0) {
            *adj_nnz = total;
            if (total > adj_cap || total > 0x7FFFFFFFll) atomicOr(status, CSGS_ST_ADJ_OVERFLOW);
        }
    }
}

// One pass: a block publishes its chunk's count and waits for the earlier chunks' before it places anything.  All blocks
// are resident; block b takes chunks b, b + grid, ... in ascending order.  Its registers decide how many blocks a compute unit holds (eight
// would need scratch memory: 0.5 us more a launch), a quarter of those is a call's (see resident_grid).
constexpr int ADJ_ONCE_BLOCKS = 7;   // per compute unit
__global__ __launch_bounds__(256, ADJ_ONCE_BLOCKS) void adj_once(AdjGraph g, const int64_t *__restrict__ meta, uint64_t *__restrict__ epoch,
                                                uint64_t *__restrict__ ts_mem, int64_t chunk_cap, const int2 *__restrict__ bound_note,
                                                int32_t *__restrict__ adj_rowptr, int32_t *__restrict__ adj_col,
                                                float *__restrict__ adj_val, int64_t adj_cap, int64_t *__restrict__ adj_nnz,
                                                int32_t *__restrict__ status, RemoteArgs rem, NextRows nxt, InstStride is)
{
    is = at_instance(is);
    epoch = inst_ptr(epoch, is.ws); status = inst_ptr(status, is.buf);
    if (adj_leading_blocks(rem, nxt, epoch, status, is, blockIdx.x)) return;
    meta = inst_ptr(meta, is.ws); g.eoff = inst_ptr(g.eoff, is.ws); g.rowstart = inst_ptr(g.rowstart, is.ws);
    g.rank = inst_ptr(g.rank, is.ws); g.member = inst_ptr(g.member, is.ws); g.pdbl = inst_ptr(g.pdbl, is.ws);
    ts_mem = inst_ptr(ts_mem, is.ws); bound_note = inst_ptr(bound_note, is.ws);
    adj_rowptr = inst_ptr(adj_rowptr, is.buf); adj_col = inst_ptr(adj_col, is.buf); adj_val = inst_ptr(adj_val, is.buf);
    adj_nnz = inst_ptr(adj_nnz, is.buf);
    const int64_t bid = (int64_t)blockIdx.x - rem.blocks - nxt.blocks;
    const int64_t n_bids = (int64_t)gridDim.x - rem.blocks - nxt.blocks;
    __shared__ AdjChunk s;
    __shared__ unsigned long long s_lb[1];
    ChunkRows rows = chunk_rows(bound_note, bid, bid + 1);   // (the grid stays within the notes; on its way beside the counts)
    const TileState<1> ts(ts_mem, chunk_cap, wait_limit(epoch));
    const unsigned long long call = call_number(epoch);
    const unsigned long long tag = call_tag(call, SLOT_ADJ);
    const uint64_t rank_tag = (epoch[EPOCH_DRAW] & 0xFFFFFFFFull) << 32;
    const int32_t nS = (int32_t)meta[META_ROWS];
    const int64_t ptr_max = adj_cap < 0x7FFFFFFFll ? adj_cap : 0x7FFFFFFFll;   // (see adj_place)
    int64_t E = meta[META_EDGES];
    int64_t n_chunks = (E + EDGE_TILE - 1) / EDGE_TILE;
    const bool overflow = n_chunks > chunk_cap;
    if (overflow) { E = 0; n_chunks = 0; }
    if (n_chunks == 0) {
        if (bid == 0) {
            for (int32_t a = threadIdx.x; a <= nS; a += blockDim.x) adj_rowptr[a] = 0;
            if (threadIdx.x == 0) {
                *adj_nnz = 0;
                if (overflow) atomicOr(status, CSGS_ST_EDGE_OVERFLOW);
                epoch[EPOCH_CALLS] = call;
            }
        }
        return;
    }
    for (int64_t t = bid; t < n_chunks; t += n_bids) {
        const int64_t c0 = t * EDGE_TILE;
        const int64_t c1 = (c0 + EDGE_TILE < E) ? c0 + EDGE_TILE : E;
        int32_t rk[4], at[4];
        int64_t ea[4];
        float pv[4];
        if (t != bid) rows = chunk_rows(bound_note, t, t + 1);
        int32_t off = adj_chunk(s, g, nS, c0, c1, rank_tag, rows, rk, ea);
        const int32_t tile_cnt = s.pre[EDGE_TILE / 64];
        unsigned long long local[1] = {(unsigned long long)tile_cnt}, excl[1];
        lookback_publish<1>(ts, tag, t, local);
        adj_values(s, g, rk, ea, pv, at);   // does not depend on the prefix: fetch and divide while it is resolved
        lookback_resolve<1>(ts, tag, t, n_chunks, local, excl, s_lb, status);
        const int64_t base = (int64_t)excl[0];
        // row pointers of the rows that start inside this chunk (the last one's: or behind it): kept edges before the row start
        const int32_t len = (int32_t)(c1 - c0);
        const bool last = t == n_chunks - 1;
        for (int32_t a = rows.first + (int32_t)threadIdx.x; a < rows.end;) {
            if (off >= 0 && (off < len || last)) {
                const int64_t v = base + (off < len ? kept_before(s, off) : tile_cnt);
                adj_rowptr[a] = (int32_t)(v < ptr_max ? v : ptr_max);
            }
            a += (int32_t)blockDim.x;
            if (a < rows.end) off = (int32_t)(g.eoff[a] - c0);   // (a row behind the first one starts inside the chunk or at its end)
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (rk[k] > 0 && base + at[k] < adj_cap) {
                adj_col[base + at[k]] = rk[k] - 1;
                adj_val[base + at[k]] = pv[k];
            }
        if (last) {
            // rows behind the last one with edges, and the end pointer
            const int64_t total = base + tile_cnt;
            const int32_t clamp = (int32_t)(total < ptr_max ? total : ptr_max);
            for (int64_t a = (rows.end < 0 ? 0 : rows.end) + (int64_t)threadIdx.x; a <= nS; a += blockDim.x) adj_rowptr[a] = clamp;
            if (threadIdx.x == 0) {
                *adj_nnz = total;
                if (total > adj_cap || total > 0x7FFFFFFFll) atomicOr(status, CSGS_ST_ADJ_OVERFLOW);
                epoch[EPOCH_CALLS] = call;  // last kernel of the call, last chunk: all chunk owners have read the counter
            }
        }
    }
}

}  // namespace csgs
using namespace csgs;

extern "C" int csgs_draw_nodes(int64_t n_nodes, const int32_t *cand_id, const uint64_t *cdf, int64_t cand_cap,
                               const csgs_prob_stats *stats, int32_t B, uint64_t seed, uint64_t iter,
                               const uint64_t *iter_dev, uint32_t layer, int32_t *S_next, int32_t *mult, float *p_incl,
                               int32_t *n_next, csgs_workspace *ws, int32_t *status, void *stream)
{
    if (n_nodes <= 0 || n_nodes > 0x7FFFFFFFll || !cand_id || !cdf || cand_cap <= 0 || !stats || B <= 0 || !S_next ||
        !mult || !p_incl || !n_next || !ws || !status)
        return CSGS_EINVAL;
    Workspace w;
    const int rc = open_workspace(ws, n_nodes, 1, B, &w);
    if (rc != CSGS_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    if (cand_cap > n_nodes) cand_cap = n_nodes;  // there are never more candidates than nodes

    const InstGrid dg = inst_grid(w, ((int64_t)B + DRAW_BLOCK - 1) / DRAW_BLOCK, DRAW_BLOCK);
    CSGS_LAUNCH(K_DRAW, draw, dg.grid, dim3(DRAW_BLOCK), st, cdf, stats,
                cand_cap, B, (uint32_t)seed, (uint32_t)(seed >> 32), iter, iter_dev, layer, w.hit, w.cbitmap[0], w.cbitmap[1], w.epoch, w.rank,
                w.member, n_nodes, dg.is);
    CSGS_LAUNCH_CHECK();
    const int64_t cap_words = (cand_cap + 63) / 64;
    const int64_t hit_blocks = (cap_words + HIT_MIN_WORDS - 1) / HIT_MIN_WORDS;
    const InstGrid hg = inst_grid(w, hit_blocks < HIT_GRID ? hit_blocks : HIT_GRID, 256);
    CSGS_LAUNCH(K_HITS, hits, hg.grid, dim3(256), st, cand_id,
                cdf, stats, cand_cap, n_nodes, B, w.epoch, w.hit, w.cbitmap[0], w.cbitmap[1], w.rank, w.member, S_next, mult, p_incl,
                w.pdbl, n_next, w.hit_ts, status, hg.is);
    CSGS_LAUNCH_CHECK();
    ws->has_draw = 1;
    ws->draw_B = B;
    ws->has_next = 0;   // offsets prepared for an earlier node set are void
    return CSGS_OK;
}

// rows == nullptr: reuse the row offsets that csgs_build_probs left in the workspace for the same rows
static int sampled_adjacency_impl(const csgs_graph *g, const int32_t *rows, int32_t n_rows, const int32_t *n_rows_dev,
                                  bool reuse_offsets,
                                  int32_t *adj_rowptr, int32_t *adj_col, float *adj_val, int64_t adj_cap,
                                  int64_t *adj_nnz, csgs_workspace *ws, int32_t *status, const RemoteArgs &rem,
                                  const int32_t *S_next, const int32_t *n_next, void *stream)
{
    if (!g || !g->rowptr || !g->colidx || !g->val || g->n_nodes <= 0 || g->n_nodes > 0x7FFFFFFFll || (!rows && !reuse_offsets) ||
        n_rows <= 0 ||
        !adj_rowptr || !adj_col || !adj_val || adj_cap <= 0 || !adj_nnz || !ws || !status)
        return CSGS_EINVAL;
    if (!ws->has_draw) return CSGS_EINVAL;  // no csgs_draw_nodes has run on this workspace
    Workspace w;
    const int rc = open_workspace(ws, g->n_nodes, n_rows, ws->draw_B, &w);
    if (rc != CSGS_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const RowOffsets &cur = w.rows[ws->rows_buf & 1];
    if (!reuse_offsets) {
        const int rc2 = launch_row_prefix(g->rowptr, g->n_nodes, rows, n_rows, n_rows_dev, w, cur, status, st);
        if (rc2 != CSGS_OK) return rc2;
    }
    // prepare the other set of row offsets for the new node set, if it fits there
    NextRows nxt{};
    if (S_next && ws->draw_B <= ws->nS_max) {
        const RowOffsets &o = w.rows[(ws->rows_buf & 1) ^ 1];
        nxt = NextRows{g->rowptr, g->n_nodes, S_next, n_next, ws->draw_B, w.rp_ts, w.rp_tiles, o.eoff, o.rowstart, o.meta,
                       o.bound_note, w.chunk_cap * EDGE_TILE, (int32_t)((ws->draw_B + ROW_TILE - 1) / ROW_TILE)};
    }
    ws->has_next = nxt.blocks > 0;
    // The number of chunks is known on the device only.  Rows of the graph's mean degree are a guess that hubs can exceed
    // many times over: it picks the path, and may ask for more blocks but not for fewer than the device holds (those without a
    // chunk leave at once; two per compute unit over several instances, where they are not free) unless the workspace
    // describes fewer chunks.  (us, grid by the mean degree / as here: 256 rows of 5000 edges, mean degree 8, one pass 317 / 26,
    // eight instances of that 324 / 122; the 8192 rows of most edges in 2.4 M, 21 M edges of them, two passes 638 / 245.)
    const double guess = (double)n_rows * ((double)g->nnz / (double)g->n_nodes) / EDGE_TILE * 1.25 + 16.0;
    const int64_t expected = guess < (double)w.chunk_cap ? (int64_t)guess : w.chunk_cap;
    auto blocks = [&](int64_t grid, int64_t chunks_each) {   // at most `grid`
        const int64_t least = w.n_inst == 1 ? grid : 512 / w.n_inst;
        int64_t n = (expected + chunks_each - 1) / chunks_each;
        if (n < least) n = least;
        if (n > grid) n = grid;
        const int64_t cap = (w.chunk_cap + chunks_each - 1) / chunks_each;
        return (unsigned)(n < cap ? n : cap);
    };
    const AdjGraph ag{g->colidx, g->val, g->n_nodes, g->nnz, cur.eoff, cur.rowstart, w.rank, w.member, w.pdbl};
    if (expected * w.n_inst <= (w.n_inst == 1 ? ADJ_ONCE_MAX : ADJ_ONCE_MAX_EACH)) {
        const dim3 grid_once(blocks(resident_grid(ADJ_ONCE_BLOCKS) / CALL_SEQUENCES, 1) + (unsigned)(rem.blocks + nxt.blocks), 1, (unsigned)w.n_inst);   // (its blocks wait for each other: an instance after the other)
        CSGS_LAUNCH(K_ADJ_ONCE, adj_once, grid_once, dim3(256), st, ag, cur.meta, w.epoch, w.adj_ts, w.chunk_cap, cur.bound_note,
                    adj_rowptr, adj_col, adj_val, adj_cap, adj_nnz, status, rem, nxt, inst_stride(w));
        CSGS_LAUNCH_CHECK();
        return CSGS_OK;
    }
    const unsigned mark = blocks(ADJ_MARK_GRID, 1), place = blocks(ADJ_PLACE_GRID, ADJ_PLACE_MIN);
    const InstGrid mg = inst_grid(w, mark + (int64_t)(rem.blocks + nxt.blocks), 256);
    CSGS_LAUNCH(K_ADJ_MARK, adj_mark, mg.grid, dim3(256), st, ag, cur.meta, w.epoch, w.chunk_cap, cur.bound_note, w.adj_cnt, w.stage,
                w.stage_chunks, adj_rowptr, status, rem, nxt, mg.is);
    CSGS_LAUNCH_CHECK();
    CSGS_LAUNCH(K_ADJ_PLACE, adj_place, each_instance(w, place), dim3(256), st, ag, cur.meta, w.epoch, w.chunk_cap, cur.bound_note, w.adj_cnt,
                w.stage, w.stage_chunks, adj_rowptr, adj_col, adj_val, adj_cap, adj_nnz, status, inst_stride(w));
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

extern "C" int csgs_sampled_adjacency(const csgs_graph *g, const int32_t *rows, int32_t n_rows,
                                      const int32_t *n_rows_dev, int32_t *adj_rowptr, int32_t *adj_col, float *adj_val, int64_t adj_cap, int64_t *adj_nnz,
                                      csgs_workspace *ws, int32_t *status, void *stream)
{
    return sampled_adjacency_impl(g, rows, n_rows, n_rows_dev, false, adj_rowptr, adj_col, adj_val, adj_cap, adj_nnz, ws, status,
                                  RemoteArgs{}, nullptr, nullptr, stream);
}

extern "C" int csgs_sample_layer(const csgs_graph *g, const int32_t *S, int32_t nS, const int32_t *cand_id,
                                 const uint64_t *cdf, int64_t cand_cap, const csgs_prob_stats *stats, int32_t B, uint64_t seed,
                                 uint64_t iter, const uint64_t *iter_dev, uint32_t layer, int32_t *S_next, int32_t *mult, float *p_incl,
                                 int32_t *n_next, int32_t *adj_rowptr, int32_t *adj_col, float *adj_val,
                                 int64_t adj_cap, int64_t *adj_nnz, const csgs_remote_out *remote,
                                 csgs_workspace *ws, int32_t *status, void *stream)
{
    if (!g || nS <= 0 || !adj_rowptr || !adj_col || !adj_val || adj_cap <= 0 || !adj_nnz) return CSGS_EINVAL;
    RemoteArgs rem{};
    if (remote) {
        if (!remote->remote_total || remote->local_lo > remote->local_hi ||
            (remote->per_part && (!remote->part_bounds || remote->P <= 0)))
            return CSGS_EINVAL;
        rem = RemoteArgs{S_next, n_next, remote->local_lo, remote->local_hi, remote->part_bounds,
                         remote->per_part ? remote->P : 0, remote->remote_total, remote->per_part, remote->src_row,
                         remote->remote_ids, remote_blocks(B, remote->per_part ? remote->P : 0)};
    }
    const int rc = csgs_draw_nodes(g->n_nodes, cand_id, cdf, cand_cap, stats, B, seed, iter, iter_dev, layer, S_next, mult, p_incl,
                                   n_next, ws, status, stream);
    if (rc != CSGS_OK) return rc;
    return sampled_adjacency_impl(g, S, nS, nullptr, true, adj_rowptr, adj_col, adj_val, adj_cap, adj_nnz, ws, status, rem, S_next, n_next, stream);
}

extern "C" int csgs_remote_count(const int32_t *S_next, const int32_t *n_next, int32_t local_lo, int32_t local_hi,
                                 const int32_t *part_bounds, int32_t P, int64_t *remote_total, int64_t *per_part,
                                 int32_t *src_row, int32_t *remote_ids, void *stream)
{
    if (!S_next || !n_next || local_lo > local_hi || !remote_total) return CSGS_EINVAL;
    if (per_part && (!part_bounds || P <= 0)) return CSGS_EINVAL;
    // the element count is known only on the device: 64 blocks of 256 cover the usual budgets in one sweep
    const RemoteArgs rem{S_next, n_next, local_lo, local_hi, part_bounds, per_part ? P : 0, remote_total, per_part, src_row,
                         remote_ids, 64};
    CSGS_LAUNCH(K_REMOTE_COUNT, remote_count_k, dim3(64), dim3(256), (hipStream_t)stream, rem);
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}
