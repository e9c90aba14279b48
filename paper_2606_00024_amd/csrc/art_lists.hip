// Traversal lists for the decode call (Sec. 3.4): the importance-first list
// of a policy that scores KV blocks, and the sink-preserving recency-first
// list of a policy that keeps sink tokens plus a recent window.
//
// Two launches:
//   1. block scores (importance lists only), one wavefront per KV block of a
//      (sequence, KV head) group, written as doubles:
//        key norm:    max over the block's tokens of sum_d k_d^2
//        query bound: max over the group's query heads of
//                     sum_d max(q_d * min_j k_jd, q_d * max_j k_jd)
//      Every sum runs over d = 0, 1, ..., 127 in order in fp64, on exact
//      products of bf16 values, so the scores do not depend on how the work
//      is split: equal inputs give equal bits on any implementation that
//      keeps that order.
//   2. selection, one workgroup per group: a merge sort of (score, id)
//      pairs in LDS, descending score and ascending id; the forced blocks
//      (the first sink_blocks, and the last when asked) and the best others
//      up to the budget are kept in sorted order.  Streaming lists need no
//      scores: sinks in increasing order, then the most recent blocks.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

#include "art.h"
#include "art_internal.h"

namespace art {
namespace {

constexpr int kListThreads = 1024;   // selection workgroup
constexpr int kMaxListBlocks = 8192; // blocks per sequence the selection sorts in LDS

struct ListParams {
    int32_t batch, num_q_heads, num_kv_heads, block_size, page_shift, num_pages;
    int32_t max_pages, max_blocks, max_list, sort_n;
    int64_t ks_page, ks_head, ks_tok;
    int32_t policy, score_kind, budget, sink_blocks, keep_last;
    int32_t pad;      // 1: entries past a row's length are set to -1
    int32_t packed;   // 1: the score kernels walk the blocks that hold tokens (see Walk)
    const uint16_t* q;
    const uint16_t* k;
    const int32_t* page_table;
    const int32_t* seq_lens;
    int32_t* list;
    int32_t* list_len;
    double* scores;   // [groups][max_blocks]
};

typedef unsigned int u32x4_l __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double bf16_lo(uint32_t w) { return (double)__uint_as_float(w << 16); }
__device__ __forceinline__ double bf16_hi(uint32_t w) { return (double)__uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ int seq_len_of(const ListParams& P, int b) {
    const int64_t cap = (int64_t)P.max_pages << P.page_shift;
    const int L = P.seq_lens[b];
    return L < 0 ? 0 : (int)(L > cap ? cap : L);
}


// wave-wide max of a double (exact)
__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmax(x, __shfl_xor(x, o));
    return x;
}

// A wavefront reads 64 tokens (one 16 KiB tile) of a block with coalesced
// 16-byte loads: load i of lane l holds bytes 16*(l & 15) .. +15 of token
// 4i + (l >> 4), which lies in 16-token piece i / 4 of the tile.  A piece
// never straddles a page where pages hold at least 16 tokens and blocks begin
// at multiples of 16 (WHOLE; every size that the decode call takes): one page
// id per piece then serves its four loads.  For other sizes each load looks
// up its own token's page.
constexpr int kTileLoads = 16;
constexpr int kRowPitch = 272;   // bytes per token row in the LDS tile (256 + 16 of padding)

// The score kernels are persistent: wavefront w walks the blocks w, w + W,
// ... (W = wavefronts in the grid), one 64-token tile at a time.  With up to
// kListLenCache sequences these are the blocks that hold tokens, group after
// group, so that every wavefront has the same share of them whatever the
// lengths.  (Walking groups of max_blocks and skipping the blocks past their
// sequence's end gave a wavefront the same few block indices of every group
// where W is a multiple of max_blocks: the early ones of them all, or only
// those of the longest sequences.  16 sequences of 2K to 64K tokens, 8 KV
// heads: key norm 256 -> 239 us, query bound 278 -> 253; 8 of 4K to 32K, query
// bound 69 -> 64; equal lengths 199 -> 202.)  Larger batches are walked that
// way: their lengths are in no table a wavefront can search in one step.
// The loads of the next tile are issued before the current tile is
// processed, and the page ids two tiles ahead before that, so that every
// wavefront keeps one tile of keys in flight while it computes.  Two things
// keep that overlap intact: every load is issued by every lane on every
// path (addresses are clamped instead of branched around, so the compiler
// can count the loads still in flight instead of waiting for all of them),
// and the two tile buffers swap roles in an unrolled pair of steps instead
// of being copied (a copy would wait for the next tile's loads).  The
// sequence lengths of the first kListLenCache sequences are read from LDS.
constexpr int kListLenCache = 256;

struct TilePos {
    int64_t item;   // position in the walk; >= n_items when done
    int gidx, b, kvh, blk, t0, j1;
};

// The walk's table: the lengths of the first kListLenCache sequences, and,
// when they are all of them, where each sequence's blocks start in the walk.
struct WalkTable {
    int len[kListLenCache];
    int start[kListLenCache];
};
struct Walk {
    const WalkTable* table;      // in LDS
    bool packed;                 // blocks that hold tokens only
    int64_t stride, n_items;
    int end[kListLenCache / 64]; // lane l: where the blocks of sequence l + 64 j end
};

__device__ __forceinline__ int cached_len(const ListParams& P, const Walk& W, int b) {
    return b < kListLenCache ? W.table->len[b] : seq_len_of(P, b);
}

// The first tile of the first block at or after `item` that holds tokens.
__device__ __forceinline__ TilePos first_tile(const ListParams& P, const Walk& W, int64_t item) {
    TilePos t;
    t.gidx = t.b = t.kvh = t.blk = t.t0 = 0;
    t.j1 = 1;
    if (W.packed) {
        if (item < W.n_items) {
            // the sequences whose blocks end at or before the item come before its own
            int b = 0;
#pragma unroll
            for (int j = 0; j < kListLenCache / 64; ++j) b += __popcll(__ballot(W.end[j] <= (int)item));
            b = __builtin_amdgcn_readfirstlane(b);
            const int L = __builtin_amdgcn_readfirstlane(W.table->len[b]);
            const int r = (int)item - __builtin_amdgcn_readfirstlane(W.table->start[b]);
            const int blocks = (L + P.block_size - 1) / P.block_size;
            t.b = b; t.kvh = r / blocks; t.blk = r - t.kvh * blocks;
            t.gidx = b * P.num_kv_heads + t.kvh;
            t.t0 = t.blk * P.block_size; t.j1 = min(t.t0 + P.block_size, L);
        }
        t.item = item;
        return t;
    }
    for (; item < W.n_items; item += W.stride) {
        const int gidx = (int)(item / P.max_blocks), blk = (int)(item % P.max_blocks);
        const int b = gidx / P.num_kv_heads;
        const int L = cached_len(P, W, b);
        const int j0 = blk * P.block_size;
        if (j0 < L) {
            t.gidx = gidx; t.b = b; t.kvh = gidx % P.num_kv_heads; t.blk = blk;
            t.t0 = j0; t.j1 = min(j0 + P.block_size, L);
            break;
        }
    }
    t.item = item;
    return t;
}

__device__ __forceinline__ TilePos next_tile(const ListParams& P, const Walk& W, TilePos t) {
    if (t.item >= W.n_items) return t;
    if (t.t0 + 64 < t.j1) {
        t.t0 += 64;
        return t;
    }
    return first_tile(P, W, t.item + W.stride);
}

// Page of a token of the tile's sequence.  Every lane reads a valid entry; a
// tile past the end reads the first one.
__device__ __forceinline__ int page_of(const ListParams& P, const TilePos& t, bool live, int tok) {
    const int64_t at = live ? (int64_t)t.b * P.max_pages + (tok >> P.page_shift) : 0;
    int pg = P.page_table[at];
    return pg < 0 ? 0 : (pg >= P.num_pages ? P.num_pages - 1 : pg);
}

// Page of 16-token piece (lane & 3) of the tile, in lane n (n < 4).
template <bool WHOLE>
__device__ __forceinline__ int tile_pages(const ListParams& P, const TilePos& t, int64_t n_items,
                                          int lane) {
    if constexpr (!WHOLE) return 0;
    const bool live = t.item < n_items;
    return page_of(P, t, live, live ? min(t.t0 + 16 * (lane & 3), t.j1 - 1) : 0);
}

// Rows past the tile's end read the tile's first row again, and every row
// of a tile past the end of the work reads the pool's first row: the
// callers ignore them, and they add no memory traffic beyond a line or two.
template <bool WHOLE>
__device__ __forceinline__ void load_tile(const ListParams& P, const TilePos& t, int pages, int64_t n_items,
                                          int lane, u32x4_l (&v)[kTileLoads]) {
    const int pmask = (1 << P.page_shift) - 1;
    const bool live = t.item < n_items;
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) {
        int tok = t.t0 + 4 * i + (lane >> 4);
        int pg = __builtin_amdgcn_readlane(pages, i >> 2);
        if (tok >= t.j1) {
            tok = t.t0;
            pg = __builtin_amdgcn_readlane(pages, 0);
        }
        if constexpr (!WHOLE) pg = page_of(P, t, live, tok);
        const uint16_t* row = live ? P.k + pg * P.ks_page + t.kvh * P.ks_head + (int64_t)(tok & pmask) * P.ks_tok
                                   : P.k;
        v[i] = reinterpret_cast<const u32x4_l*>(row)[lane & 15];
    }
}

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's LDS accesses are done
    __builtin_amdgcn_wave_barrier();
}

// Fills the walk's table (every thread of the workgroup takes part; a barrier
// follows) and sets up this wavefront's walk.
__device__ __forceinline__ Walk make_walk(const ListParams& P, WalkTable* table) {
    const int lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < min(P.batch, kListLenCache); i += blockDim.x) table->len[i] = seq_len_of(P, i);
    __syncthreads();
    Walk W;
    W.table = table;
    W.packed = P.packed;
    W.stride = (int64_t)gridDim.x * 4;
    W.n_items = (int64_t)P.batch * P.num_kv_heads * P.max_blocks;
    if (W.packed) {
        // every wavefront sums the sequences' blocks itself, 64 at a time
        int before = 0;
#pragma unroll
        for (int j = 0; j < kListLenCache / 64; ++j) {
            const int b = 64 * j + lane;
            W.end[j] = before;
            if (64 * j >= P.batch) continue;   // (no sequences: past every position of the walk)
            const int own = b < P.batch ? (table->len[b] + P.block_size - 1) / P.block_size * P.num_kv_heads : 0;
            int sum = own;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(sum, o);
                if (lane >= o) sum += y;
            }
            W.end[j] = before + sum;
            // (the wavefronts store the same values)
            table->start[b] = before + sum - own;
            before += __builtin_amdgcn_readlane(sum, 63);
        }
        W.n_items = before;
        __syncthreads();
    }
    return W;
}

// Walks this wavefront's tiles with the loads one tile ahead; `pre_fn(t)`
// issues the loads that the current tile's `block_fn` will need (before the
// next tile's keys, so that waiting for them does not wait for the keys),
// `tile_fn(t, v)` consumes a tile, `block_fn(t)` ends a block (after its
// last tile).
template <bool WHOLE, class PreFn, class TileFn, class BlockFn>
__device__ __forceinline__ void stream_tiles(const ListParams& P, const Walk& W, PreFn pre_fn,
                                             TileFn tile_fn, BlockFn block_fn) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t n_items = W.n_items;
    TilePos cur = first_tile(P, W, (int64_t)blockIdx.x * 4 + wave);
    if (cur.item >= n_items) return;
    TilePos nxt = next_tile(P, W, cur);
    const int pg_cur = tile_pages<WHOLE>(P, cur, n_items, lane);
    int pg_nxt = tile_pages<WHOLE>(P, nxt, n_items, lane);
    u32x4_l a[kTileLoads], b[kTileLoads];
    load_tile<WHOLE>(P, cur, pg_cur, n_items, lane, a);
    // One step: the page ids two tiles ahead, the keys of the next tile into
    // `nb`, then the current tile (in `cb`).  False once the work is done.
    auto step = [&](u32x4_l (&cb)[kTileLoads], u32x4_l (&nb)[kTileLoads]) -> bool {
        const TilePos nn = next_tile(P, W, nxt);
        const int pg_nn = tile_pages<WHOLE>(P, nn, n_items, lane);
        pre_fn(cur);
        load_tile<WHOLE>(P, nxt, pg_nxt, n_items, lane, nb);
        tile_fn(cur, cb);
        if (nxt.item != cur.item) block_fn(cur);
        if (nxt.item >= n_items) return false;
        cur = nxt;
        nxt = nn;
        pg_nxt = pg_nn;
        return true;
    };
    while (step(a, b) && step(b, a)) {
    }
}

// Lane j sums the 128 squares of token j in dimension order: the tile goes
// through LDS (64 rows per wavefront).  Each square of a bf16 value is exact
// in fp64, so the fused multiply-add rounds once per term, as the separate
// product and sum would.  Rows past the block's end hold its first row
// again (load_tile), which leaves the maximum unchanged.
constexpr int kKeyNormLds = 4 * 64 * kRowPitch;   // bytes per workgroup

template <bool WHOLE>
__global__ void __launch_bounds__(256) score_key_norm_kernel(const ListParams P) {
    extern __shared__ __align__(16) unsigned char tiles[];
    __shared__ WalkTable table;
    const Walk W = make_walk(P, &table);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned char* tile = tiles + w * 64 * kRowPitch;
    double best = -1.0;   // below any sum of squares
    stream_tiles<WHOLE>(P, W, [](const TilePos&) {},
        [&](const TilePos&, const u32x4_l (&v)[kTileLoads]) {
#pragma unroll
            for (int i = 0; i < kTileLoads; ++i)
                *reinterpret_cast<u32x4_l*>(tile + (4 * i + (lane >> 4)) * kRowPitch + 16 * (lane & 15)) = v[i];
            wave_lds_fence();
            const unsigned char* row = tile + lane * kRowPitch;
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const u32x4_l x = *reinterpret_cast<const u32x4_l*>(row + 16 * c);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double x0 = bf16_lo(x[e]), x1 = bf16_hi(x[e]);
                    s = __builtin_fma(x0, x0, s);   // dimension 8c + 2e
                    s = __builtin_fma(x1, x1, s);   // dimension 8c + 2e + 1
                }
            }
            best = fmax(best, s);
            wave_lds_fence();   // the rows are read before they are written again
        },
        [&](const TilePos& t) {
            // every lane stores the same value (no branch around the store)
            P.scores[(int64_t)t.gidx * P.max_blocks + t.blk] = wave_max(best);
            best = -1.0;
        });
}

// Lane l keeps the extremes of dimensions 8*(l & 15) .. +7 over the tokens
// its loads cover; at the end of a block the four lane rows are combined,
// the per-dimension terms of every query head go to LDS, and lane h sums
// head h's 128 terms in order.
//
// The extremes are taken on the raw bf16 words, two dimensions per
// instruction, with no conversion: a bf16 is sign and magnitude, so over a
// set of values the largest is the largest as a signed 16-bit integer when
// that one is non-negative and otherwise (all negative) the smallest as a
// signed integer; the smallest is the largest as an unsigned integer when
// any sign bit is set and otherwise the smallest as an unsigned integer.
// Four packed extremes per word (signed and unsigned, largest and
// smallest) give both.  This holds for every value but NaN (keys hold
// none) and treats -0 as the smallest negative, which changes no term:
// q * (+-0) is a zero either way and adding a zero of either sign to the
// running sum, which starts at +0, gives the same bits.  Rows past the
// block's end hold its first row again (load_tile), which changes no
// extreme.
typedef short s16x2_l __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2_l __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_smax(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2_l, a),
                                                                  __builtin_bit_cast(s16x2_l, b)));
}
__device__ __forceinline__ uint32_t pk_smin(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(s16x2_l, a),
                                                                  __builtin_bit_cast(s16x2_l, b)));
}
__device__ __forceinline__ uint32_t pk_umax(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_l, a),
                                                                  __builtin_bit_cast(u16x2_l, b)));
}
__device__ __forceinline__ uint32_t pk_umin(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_l, a),
                                                                  __builtin_bit_cast(u16x2_l, b)));
}

// The value (as a float) of the largest and the smallest bf16 of one half
// (shift 0: low, 16: high) of the four packed extremes.
__device__ __forceinline__ void half_extremes(uint32_t smax, uint32_t smin, uint32_t umax, uint32_t umin,
                                              int shift, float& lo, float& hi) {
    const uint32_t sx = (smax >> shift) & 0xffffu, sn = (smin >> shift) & 0xffffu;
    const uint32_t ux = (umax >> shift) & 0xffffu, un = (umin >> shift) & 0xffffu;
    hi = __uint_as_float((sx < 0x8000u ? sx : sn) << 16);
    lo = __uint_as_float((ux >= 0x8000u ? ux : un) << 16);
}

template <int G, bool WHOLE>
__global__ void __launch_bounds__(256) score_query_bound_kernel(const ListParams P) {
    __shared__ double terms[4][G][128];
    __shared__ WalkTable table;
    const Walk W = make_walk(P, &table);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // word e of the lane's 16 bytes: dimensions 8c + 2e (low half), 8c + 2e + 1
    uint32_t smax[4], smin[4], umax[4], umin[4];
    auto reset = [&]() {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            smax[e] = 0x80008000u; smin[e] = 0x7fff7fffu; umax[e] = 0u; umin[e] = 0xffffffffu;
        }
    };
    reset();
    // lane row r holds dimensions 8*(lane & 15) .. +7 of query heads r, r + 4, ...
    constexpr int QR = (G + 3) / 4;
    u32x4_l qw[QR];
    const int c = lane & 15, r = lane >> 4;
    stream_tiles<WHOLE>(P, W,
        [&](const TilePos& t) {
#pragma unroll
            for (int h0 = 0, u = 0; h0 < G; h0 += 4, ++u) {
                const int h = min(h0 + r, G - 1);
                qw[u] = reinterpret_cast<const u32x4_l*>(
                    P.q + ((int64_t)t.b * P.num_q_heads + t.kvh * G + h) * kHeadDim)[c];
            }
        },
        [&](const TilePos&, const u32x4_l (&v)[kTileLoads]) {
#pragma unroll
            for (int i = 0; i < kTileLoads; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    smax[e] = pk_smax(smax[e], v[i][e]); smin[e] = pk_smin(smin[e], v[i][e]);
                    umax[e] = pk_umax(umax[e], v[i][e]); umin[e] = pk_umin(umin[e], v[i][e]);
                }
            }
        },
        [&](const TilePos& t) {
            // lanes l, l ^ 16, l ^ 32, l ^ 48 hold the same dimensions
#pragma unroll
            for (int e = 0; e < 4; ++e) {
#pragma unroll
                for (int o = 16; o <= 32; o <<= 1) {
                    smax[e] = pk_smax(smax[e], (uint32_t)__shfl_xor((int)smax[e], o));
                    smin[e] = pk_smin(smin[e], (uint32_t)__shfl_xor((int)smin[e], o));
                    umax[e] = pk_umax(umax[e], (uint32_t)__shfl_xor((int)umax[e], o));
                    umin[e] = pk_umin(umin[e], (uint32_t)__shfl_xor((int)umin[e], o));
                }
            }
            float lo[8], hi[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                half_extremes(smax[e], smin[e], umax[e], umin[e], 0, lo[2 * e], hi[2 * e]);
                half_extremes(smax[e], smin[e], umax[e], umin[e], 16, lo[2 * e + 1], hi[2 * e + 1]);
            }
            // lane row r writes the terms of heads r, r + 4, ...
#pragma unroll
            for (int h0 = 0, u = 0; h0 < G; h0 += 4, ++u) {
                const int h = h0 + r;
                if (h < G) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double q0 = bf16_lo(qw[u][e]), q1 = bf16_hi(qw[u][e]);
                        terms[w][h][8 * c + 2 * e] = fmax(q0 * (double)lo[2 * e], q0 * (double)hi[2 * e]);
                        terms[w][h][8 * c + 2 * e + 1] = fmax(q1 * (double)lo[2 * e + 1], q1 * (double)hi[2 * e + 1]);
                    }
                }
            }
            wave_lds_fence();
            double s = -INFINITY;
            if (lane < G) {
                s = 0.0;
                for (int d = 0; d < 128; ++d) s = s + terms[w][lane][d];
            }
            P.scores[(int64_t)t.gidx * P.max_blocks + t.blk] = wave_max(s);
            wave_lds_fence();   // the terms are read before the next block writes them
            reset();
        });
}

// A persistent launch of 256-thread workgroups: as many as are resident at
// once (never more than one wavefront per work item), so that no workgroup
// waits for another to finish before it starts its share.  With `spread`,
// four times as many once a wavefront would have 32 tiles or more: the chip
// hands the shares out as others end, which evens out CUs that run ahead
// (key norm of 4 x 128K 203 -> 193 us, 1 x 512K 198 -> 193, 16 ragged
// sequences of up to 64K 241 -> 234; with 16 tiles each 103 -> 104).  The query
// bound's wavefronts cost more to start: 204 -> 213 us on the first.
template <class Kernel>
hipError_t launch_persistent(Kernel kernel, int64_t items, size_t lds, hipStream_t stream, const ListParams& P,
                             bool spread = false) {
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    const int64_t resident = (int64_t)cus * per_cu, tiles = items * ((P.block_size + 63) / 64);
    const int64_t grid = std::min<int64_t>((items + 3) / 4, spread && tiles >= 32 * 4 * resident ? 4 * resident : resident);
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), lds, stream, P);
    return hipGetLastError();
}

// The value that lane (lane ^ S) holds, S one of 1, 2, 4, 8, 16, 32, by
// the cross-lane moves of the vector ALU instead of a round trip through
// the LDS unit: quad permutes for 1 and 2, rotations within a row of 16
// lanes for 4 and 8 (row_ror:n hands lane i the value of lane i - n of
// its row), and the swaps of 16- and 32-lane halves for 16 and 32.
template <int S>
__device__ __forceinline__ int xor_lane(int x) {
    const int lane = threadIdx.x & 63;
    if constexpr (S == 1) {
        return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
    } else if constexpr (S == 2) {
        return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
    } else if constexpr (S == 4) {
        const int from_above = __builtin_amdgcn_mov_dpp(x, 0x12C, 0xf, 0xf, false);   // row_ror:12
        const int from_below = __builtin_amdgcn_mov_dpp(x, 0x124, 0xf, 0xf, false);   // row_ror:4
        return (lane & 4) ? from_below : from_above;
    } else if constexpr (S == 8) {
        return __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, false);  // row_ror:8
    } else if constexpr (S == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (lane & 16) ? r[0] : r[1];
    } else {
        static_assert(S == 32, "a power of two up to 32");
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (lane & 32) ? r[0] : r[1];
    }
}

template <int S>
__device__ __forceinline__ double xor_lane(double x) {
    const long long w = __double_as_longlong(x);
    const int lo = xor_lane<S>((int)(w & 0xffffffffll)), hi = xor_lane<S>((int)(w >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// a before b: larger score, then smaller id
__device__ __forceinline__ bool before(double sa, int ia, double sb, int ib) {
    return sa > sb || (sa == sb && ia < ib);
}

// exclusive prefix sum of one int per thread over the workgroup
__device__ int block_exclusive_scan(int v, int* scratch, int& total) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) scratch[w] = incl;
    __syncthreads();
    if (w == 0) {
        const int nw = kListThreads / 64;
        int x = lane < nw ? scratch[lane] : 0;
        int xi = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(xi, o);
            if (lane >= o) xi += y;
        }
        if (lane < nw) scratch[lane] = xi - x;   // exclusive offset of wave `lane`
        if (lane == nw - 1) scratch[nw] = xi;    // total
    }
    __syncthreads();
    const int r = scratch[w] + incl - v;
    total = scratch[kListThreads / 64];
    __syncthreads();
    return r;
}

// One lane's element (k, i) at position pos through the bitonic stages
// with strides S, S/2, ..., 1 of a run of `size` positions: the lower
// position of each pair keeps whichever element comes first in a run that
// puts "before" first (up), the upper one the other; the other runs the
// other way round.
template <int S>
__device__ __forceinline__ void register_stages(double& k, int& i, bool up, int lane) {
    const double pk = xor_lane<S>(k);
    const int pi = xor_lane<S>(i);
    const bool lower = (lane & S) == 0;
    if ((lower == up) != before(k, i, pk, pi)) {
        k = pk;
        i = pi;
    }
    if constexpr (S > 1) register_stages<S / 2>(k, i, up, lane);
}

// One round of a merge sort over the first `total` positions: neighbouring
// runs of `run` sorted elements become runs of twice that.  An element's
// place is its index in its own run plus the number of elements of the
// neighbouring run that come before it, found by bisection; all places are
// known before any element moves.  The elements are in id order before
// the first round, so that all ids of the lower run are the smaller ones: equal scores are told
// apart by which run is which, and the bisection reads no ids.  PER elements
// per thread.  (A bitonic network over LDS took 45 barrier phases of
// compare-and-exchange for 2048 blocks, 20 us, all of it issue on one CU; the
// bisections are 45 dependent LDS reads.)
template <int PER>
__device__ void merge_round(double* key, int* id, int total, int run) {
    const int tid = threadIdx.x;
    double k[PER];
    int i[PER], at[PER];
    bool ties[PER];   // an equal score of the neighbouring run comes before it
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int p = min(tid + u * kListThreads, total - 1);
        k[u] = key[p];
        i[u] = id[p];
        at[u] = (p & ~(run - 1)) ^ run;   // the neighbouring run, then the place in it
        ties[u] = (p & run) != 0;
    }
    auto precedes = [&](double other, int u) { return other > k[u] || (ties[u] && other == k[u]); };
    for (int step = run >> 1; step >= 1; step >>= 1)
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (precedes(key[at[u] + step - 1], u)) at[u] += step;
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (precedes(key[at[u]], u)) ++at[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int p = tid + u * kListThreads;
        if (p < total) {
            const int own = p & ~(run - 1);
            const int to = (own & ~run) + (p - own) + (at[u] - (own ^ run));
            key[to] = k[u];
            id[to] = i[u];
        }
    }
    __syncthreads();
}

// Blocks that can be on the list, in id order, into key[] and id[]; returns
// how many (n, and nothing written, if that would be all of them).  The best
// `need` blocks and the forced ones hold every entry of the list.  A
// histogram of the scores' leading bits below the highest score (as ordered
// integers, 128 bins per octave, the last one open) gives a bin at or above
// which at least `need` blocks lie; equal scores share a bin, and a higher
// score never has a later one.  What bounds the selection is its sorting on one
// CU, in steps of powers of two, so it pays where what is kept is sorted in a
// smaller one: a third of the blocks or fewer, of more than 1024 (up to 1024
// blocks are sorted in 9 us).  A quarter of 1088, 2048, 4096, 8192 blocks: 18.1
// -> 12.7 us, 18.7 -> 15.2, 35.0 -> 23.6, 72 -> 46; a third 18.1 -> 12.5, 18.7
// -> 15.3, 35.2 -> 24.8, 72 -> 43; a sixteenth of 8192 72 -> 20; but a half
// 18.1 -> 14.5, 18.7 -> 22.8, 34.6 -> 39.0, 72 -> 79.
constexpr int kFilterBlocks = 1024;
constexpr int kFilterShift = 45;
__device__ int keep_candidates(const double* sc, int n, int ns, bool last, int need, double* key, int* id,
                               int* scratch) {
    constexpr int kPer = kMaxListBlocks / kListThreads;
    const int tid = threadIdx.x, lane = tid & 63;
    int* bins = reinterpret_cast<int*>(key);   // one per thread; key[] holds more than kFilterBlocks entries
    unsigned long long* top = reinterpret_cast<unsigned long long*>(id);
    bins[tid] = 0;
    if (tid == 0) *top = 0;
    // consecutive blocks p0 .. p0 + per - 1 of each thread
    const int per = (n + kListThreads - 1) / kListThreads, p0 = tid * per;
    double s[kPer];
    unsigned long long u[kPer], best = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        const int p = p0 + e;
        s[e] = e < per && p < n ? sc[p] : -INFINITY;
        if (!(s[e] == s[e])) s[e] = -INFINITY;
        const unsigned long long w = (unsigned long long)__double_as_longlong(s[e] + 0.0);   // (-0 to +0)
        u[e] = (long long)w < 0 ? ~w : w | (1ull << 63);
        best = max(best, u[e]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) best = max(best, (unsigned long long)__shfl_xor((long long)best, o));
    __syncthreads();
    if (lane == 0) atomicMax(top, best);
    __syncthreads();
    best = *top >> kFilterShift;
    int bin[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        bin[e] = (int)min((unsigned long long)(kListThreads - 1), best - (u[e] >> kFilterShift));
        if (e < per && p0 + e < n) atomicAdd(&bins[bin[e]], 1);
    }
    __syncthreads();
    const int own = bins[tid];
    int total;
    const int above = block_exclusive_scan(own, scratch, total);
    // (the scan's last barrier is behind every read of the bins and the top)
    if (above < need && above + own >= need) *id = tid;
    __syncthreads();
    const int at = *id;
    __syncthreads();
    int cnt = 0;
    auto wanted = [&](int e) {
        const int p = p0 + e;
        return e < per && p < n && (bin[e] <= at || p < ns || (last && p == n - 1));
    };
#pragma unroll
    for (int e = 0; e < kPer; ++e) cnt += wanted(e) ? 1 : 0;
    int pos = block_exclusive_scan(cnt, scratch, total);
    if (total < n) {
#pragma unroll
        for (int e = 0; e < kPer; ++e)
            if (wanted(e)) {
                key[pos] = s[e];
                id[pos++] = p0 + e;
            }
    }
    __syncthreads();
    return total;
}

// FILTER: rows may hold more than kFilterBlocks blocks (without that code the
// selection of up to 1024 blocks takes 8.8 us in place of 9.4).
template <bool FILTER>
__global__ void __launch_bounds__(kListThreads) select_kernel(const ListParams P) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int gidx = blockIdx.x, tid = threadIdx.x;
    const int b = gidx / P.num_kv_heads;
    const int L = seq_len_of(P, b);
    const int n = L > 0 ? (L + P.block_size - 1) / P.block_size : 0;
    int32_t* out = P.list + (int64_t)gidx * P.max_list;
    if (P.policy == ART_LIST_STREAMING) {
        const int ns = min(P.sink_blocks, n);
        const int nr = min(P.budget, n - ns);
        for (int i = tid; i < ns + nr; i += kListThreads) out[i] = i < ns ? i : n - 1 - (i - ns);
        if (P.pad)
            for (int i = ns + nr + tid; i < P.max_list; i += kListThreads) out[i] = -1;
        if (tid == 0) P.list_len[gidx] = ns + nr;
        return;
    }
    // forced blocks and the budget for the others
    const int ns = min(P.sink_blocks, n);
    const int nf = ns + ((P.keep_last && n > 0 && n - 1 >= ns) ? 1 : 0);
    const int others = max(0, P.budget - nf);
    // importance: sort (score, id) pairs of blocks 0..n-1, or of those of them
    // that can be kept, into descending score, ties by ascending id.  The
    // elements that fill the sorted range up to a power of two come after
    // them all and have ids of their own, and so do NaN scores' (unspecified,
    // but the order must be total).
    double* key = reinterpret_cast<double*>(lds);
    int* id = reinterpret_cast<int*>(lds + (size_t)P.sort_n * sizeof(double));
    int* scratch = id + P.sort_n;
    const double* sc = P.scores + (int64_t)gidx * P.max_blocks;
    int m = n;
    if constexpr (FILTER) {
        const int need = max(1, max(P.budget, nf));
        if (n > kFilterBlocks && need <= n / 3) m = keep_candidates(sc, n, ns, P.keep_last != 0, need, key, id, scratch);
    }
    const bool filtered = FILTER && m < n;
    int N = 64;
    while (N < m) N <<= 1;
    // Runs of 64 first, in registers: each wavefront takes whole segments
    // (lane l holds position 64 s + l) through the bitonic stages, exchanging
    // with lane l ^ stride (xor_lane).
    const int wave = tid >> 6, lane = tid & 63;
    for (int seg = wave; seg * 64 < N; seg += kListThreads / 64) {
        const int pos = seg * 64 + lane;
        double k = -INFINITY;
        int i = kMaxListBlocks + pos;   // (past every block's id)
        if (pos < m) {
            k = filtered ? key[pos] : sc[pos];
            i = filtered ? id[pos] : pos;
        }
        if (!(k == k)) k = -INFINITY;
        register_stages<1>(k, i, (lane & 2) == 0, lane);
        register_stages<2>(k, i, (lane & 4) == 0, lane);
        register_stages<4>(k, i, (lane & 8) == 0, lane);
        register_stages<8>(k, i, (lane & 16) == 0, lane);
        register_stages<16>(k, i, (lane & 32) == 0, lane);
        register_stages<32>(k, i, true, lane);
        key[pos] = k;
        id[pos] = i;
    }
    __syncthreads();
    for (int run = 64; run < N; run <<= 1) {
        switch (N / kListThreads) {
            case 8: merge_round<8>(key, id, N, run); break;
            case 4: merge_round<4>(key, id, N, run); break;
            case 2: merge_round<2>(key, id, N, run); break;
            default: merge_round<1>(key, id, N, run); break;
        }
    }
    // each thread takes a run of consecutive sorted positions
    const int per = (N + kListThreads - 1) / kListThreads;
    const int p0 = tid * per;
    int cnt_other = 0;
    for (int p = p0; p < min(p0 + per, m); ++p) {
        const int i = id[p];
        const bool forced = i < ns || (P.keep_last && i == n - 1);
        cnt_other += forced ? 0 : 1;
    }
    int tot;
    int rank_other = block_exclusive_scan(cnt_other, scratch, tot);
    int cnt_sel = 0;
    {
        int r = rank_other;
        for (int p = p0; p < min(p0 + per, m); ++p) {
            const int i = id[p];
            const bool forced = i < ns || (P.keep_last && i == n - 1);
            if (forced) ++cnt_sel;
            else { if (r < others) ++cnt_sel; ++r; }
        }
    }
    int total_sel;
    int pos = block_exclusive_scan(cnt_sel, scratch, total_sel);
    {
        int r = rank_other;
        for (int p = p0; p < min(p0 + per, m); ++p) {
            const int i = id[p];
            const bool forced = i < ns || (P.keep_last && i == n - 1);
            bool take = forced;
            if (!forced) { take = r < others; ++r; }
            if (take) out[pos++] = i;
        }
    }
    if (P.pad)
        for (int i = total_sel + tid; i < P.max_list; i += kListThreads) out[i] = -1;
    if (tid == 0) P.list_len[gidx] = total_sel;
}

template <bool WHOLE>
hipError_t launch_scores(const art_decode_shape* s, const art_list_opts* o, const ListParams& P, hipStream_t stream) {
    const int64_t items = (int64_t)P.batch * P.num_kv_heads * P.max_blocks;
    if (o->score_kind == ART_SCORE_KEY_NORM)
        return launch_persistent(score_key_norm_kernel<WHOLE>, items, kKeyNormLds, stream, P, true);
    switch (s->num_q_heads / s->num_kv_heads) {
        case 1: return launch_persistent(score_query_bound_kernel<1, WHOLE>, items, 0, stream, P);
        case 2: return launch_persistent(score_query_bound_kernel<2, WHOLE>, items, 0, stream, P);
        case 4: return launch_persistent(score_query_bound_kernel<4, WHOLE>, items, 0, stream, P);
        case 8: return launch_persistent(score_query_bound_kernel<8, WHOLE>, items, 0, stream, P);
        default: return launch_persistent(score_query_bound_kernel<16, WHOLE>, items, 0, stream, P);
    }
}

int ilog2_exact(int v) {
    int s = 0;
    while ((1 << s) < v) ++s;
    return (1 << s) == v ? s : -1;
}

art_status check_list(const art_decode_shape* s, const art_list_opts* o, int& max_blocks, int& sort_n) {
    if (!s || !o) return ART_ERR_INVALID_ARG;
    if (s->batch < 0 || s->num_kv_heads <= 0 || s->num_q_heads <= 0 ||
        s->num_q_heads % s->num_kv_heads != 0 || s->block_size <= 0 || s->page_size <= 0 ||
        s->num_pages <= 0 || s->max_pages_per_seq <= 0 || s->max_blocks_per_list <= 0 ||
        s->list_per_head != 1 || s->k_stride_page < 0 || s->k_stride_head < 0 || s->k_stride_token < 0)
        return ART_ERR_INVALID_ARG;
    if ((o->policy != ART_LIST_IMPORTANCE && o->policy != ART_LIST_STREAMING) || o->budget < 0 ||
        o->sink_blocks < 0 || (o->keep_last != 0 && o->keep_last != 1) ||
        (o->policy == ART_LIST_IMPORTANCE && o->score_kind != ART_SCORE_KEY_NORM &&
         o->score_kind != ART_SCORE_QUERY_BOUND))
        return ART_ERR_INVALID_ARG;
    const int g = s->num_q_heads / s->num_kv_heads;
    if (s->head_dim != kHeadDim || ilog2_exact(s->page_size) < 0) return ART_ERR_UNSUPPORTED;
    if (o->policy == ART_LIST_IMPORTANCE && o->score_kind == ART_SCORE_QUERY_BOUND &&
        g != 1 && g != 2 && g != 4 && g != 8 && g != 16)
        return ART_ERR_UNSUPPORTED;
    const int64_t mb = ((int64_t)s->max_pages_per_seq * s->page_size + s->block_size - 1) / s->block_size;
    if (mb > kMaxListBlocks) return ART_ERR_UNSUPPORTED;
    max_blocks = (int)mb;
    sort_n = 64;
    while (sort_n < max_blocks) sort_n <<= 1;
    // the longest list this call can write must fit a row
    int64_t longest;
    if (o->policy == ART_LIST_STREAMING) {
        longest = std::min<int64_t>(mb, (int64_t)o->sink_blocks + o->budget);
    } else {
        const int64_t forced = std::min<int64_t>(mb, o->sink_blocks) + (o->keep_last ? 1 : 0);
        longest = std::min<int64_t>(mb, std::max<int64_t>(o->budget, forced));
    }
    if (longest > s->max_blocks_per_list) return ART_ERR_INVALID_ARG;
    return ART_OK;
}

}  // namespace
}  // namespace art

namespace {

art_status build_list(const art_decode_shape* shape, const art_list_opts* opts, const void* q,
                      const void* k_cache, const int32_t* page_table, const int32_t* seq_lens,
                      int32_t* block_list, int32_t* block_list_len, double* block_scores,
                      void* workspace, size_t workspace_bytes, bool pad, hipStream_t stream) {
    using namespace art;
    int mb = 0, sn = 0;
    art_status st = check_list(shape, opts, mb, sn);
    if (st != ART_OK) return st;
    if (shape->batch == 0) return ART_OK;
    const bool importance = opts->policy == ART_LIST_IMPORTANCE;
    if (!seq_lens || !block_list || !block_list_len) return ART_ERR_INVALID_ARG;
    if (importance && (!k_cache || !page_table)) return ART_ERR_INVALID_ARG;
    if (importance && opts->score_kind == ART_SCORE_QUERY_BOUND && !q) return ART_ERR_INVALID_ARG;
    if (importance && (((uintptr_t)k_cache | (uintptr_t)(q ? q : k_cache)) % 16 ||
                       shape->k_stride_token % 8 || shape->k_stride_head % 8 || shape->k_stride_page % 8))
        return ART_ERR_UNSUPPORTED;
    const size_t need = (size_t)shape->batch * shape->num_kv_heads * mb * sizeof(double);
    double* scores = block_scores;
    if (importance && !scores) {
        if (!workspace || workspace_bytes < need) return ART_ERR_WORKSPACE_TOO_SMALL;
        if ((uintptr_t)workspace % 8) return ART_ERR_INVALID_ARG;
        scores = static_cast<double*>(workspace);
    }
    ListParams P;
    memset(&P, 0, sizeof P);
    P.batch = shape->batch;
    P.num_q_heads = shape->num_q_heads;
    P.num_kv_heads = shape->num_kv_heads;
    P.block_size = shape->block_size;
    P.page_shift = ilog2_exact(shape->page_size);
    P.num_pages = shape->num_pages;
    P.max_pages = shape->max_pages_per_seq;
    P.max_blocks = mb;
    P.max_list = shape->max_blocks_per_list;
    P.sort_n = sn;
    P.ks_page = shape->k_stride_page;
    P.ks_head = shape->k_stride_head;
    P.ks_tok = shape->k_stride_token;
    P.policy = opts->policy;
    P.score_kind = opts->score_kind;
    P.budget = opts->budget;
    P.sink_blocks = opts->sink_blocks;
    P.keep_last = opts->keep_last;
    P.pad = pad ? 1 : 0;
    // the walk's positions are 32-bit (the stride is added to the last one)
    P.packed = shape->batch <= kListLenCache && (int64_t)shape->batch * shape->num_kv_heads * mb < (1 << 30);
    P.q = static_cast<const uint16_t*>(q);
    P.k = static_cast<const uint16_t*>(k_cache);
    P.page_table = page_table;
    P.seq_lens = seq_lens;
    P.list = block_list;
    P.list_len = block_list_len;
    P.scores = scores;
    const int groups = shape->batch * shape->num_kv_heads;
    if (importance && (int64_t)groups * mb > 0) {
        const bool whole = shape->page_size >= 16 && shape->block_size % 16 == 0;
        if ((whole ? launch_scores<true>(shape, opts, P, stream) : launch_scores<false>(shape, opts, P, stream)) != hipSuccess)
            return ART_ERR_HIP;
    }
    const size_t lds = importance ? (size_t)sn * (sizeof(double) + sizeof(int)) +
                                        (kListThreads / 64 + 1) * sizeof(int)
                                  : 0;
    auto select = importance && mb > kFilterBlocks ? select_kernel<true> : select_kernel<false>;
    hipLaunchKernelGGL(select, dim3((unsigned)groups), dim3(kListThreads), lds, stream, P);
    return hipGetLastError() == hipSuccess ? ART_OK : ART_ERR_HIP;
}
}  // namespace

extern "C" {

size_t art_block_list_workspace_bytes(const art_decode_shape* shape, const art_list_opts* opts,
                                      int32_t* status) {
    int mb = 0, sn = 0;
    const art_status st = art::check_list(shape, opts, mb, sn);
    if (status) *status = st;
    if (st != ART_OK) return 0;
    return (size_t)shape->batch * shape->num_kv_heads * mb * sizeof(double);
}

art_status art_build_block_list(const art_decode_shape* shape, const art_list_opts* opts,
                                const void* q, const void* k_cache, const int32_t* page_table,
                                const int32_t* seq_lens, int32_t* block_list,
                                int32_t* block_list_len, double* block_scores, void* workspace,
                                size_t workspace_bytes, hipStream_t stream) {
    return build_list(shape, opts, q, k_cache, page_table, seq_lens, block_list, block_list_len,
                      block_scores, workspace, workspace_bytes, false, stream);
}

art_status art_build_block_list_padded(const art_decode_shape* shape, const art_list_opts* opts,
                                       const void* q, const void* k_cache,
                                       const int32_t* page_table, const int32_t* seq_lens,
                                       int32_t* block_list, int32_t* block_list_len,
                                       double* block_scores, void* workspace,
                                       size_t workspace_bytes, hipStream_t stream) {
    return build_list(shape, opts, q, k_cache, page_table, seq_lens, block_list, block_list_len,
                      block_scores, workspace, workspace_bytes, true, stream);
}

}  // extern "C"
