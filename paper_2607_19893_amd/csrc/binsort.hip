// Rendering phase, part 1: duplicate visible primitives per touched tile and
// order the pairs by (tile, depth, primitive id).
//
// Instead of one wide radix sort over 64-bit (tile, depth) keys:
//   1. every visible primitive's tile pairs are emitted in visible-set order
//      (ascending ids), each primitive's rectangle row-major, so a primitive's
//      pairs are contiguous ("emission order"); each emission block also
//      counts its pairs per tile in LDS and adds the non-zero counts to the
//      per-tile totals (one device atomic per distinct tile of the block);
//   2. one workgroup turns the totals into the tile ranges and the dispatch
//      order (tiles by a code of their pair count, the longest first: a
//      stable counting sort over 256 codes);
//   3. the pairs are placed in their tile's range: each block ranks its pairs
//      per tile in LDS and claims one run of slots per distinct tile from the
//      tile's cursor (a device atomic), so the order of a tile's pairs inside
//      its range depends on scheduling;
//   4. each tile's segment is sorted by (depth bits, emission position), tiles
//      taken in the dispatch order by a persistent grid: a wave sorts a tile of
//      fewer than 512 pairs in registers (256 where the tiles are few), a workgroup
//      one of up to 2048 (its waves in registers, merges across waves through LDS), two exact runs
//      in LDS merged by rank up to 4096, and a network in global memory beyond.
//      The key is unique per pair, so the result does not depend on the order
//      step 3 left; emission positions grow with the primitive id inside a
//      tile, so this is exactly the (tile, depth bits, id) order.
// The per-tile kernels that follow (this sort, the forward and backward
// raster) end when their longest tile ends; taking the longest first lets
// the short ones fill in beside it instead of after it.
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace gsmi {

namespace {

// Tile counters per LDS histogram pass of the emission and placement blocks
// (32 KB); a block whose pairs span more tiles takes several passes over its keys.
constexpr uint32_t kTileChunk = 8192;

// Lanes of a wave whose digit equals this lane's digit (a 64-lane match built
// from one ballot per digit bit), restricted to the valid lanes.
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid, int nbits) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        peers &= bit ? bb : ~bb;
    }
    return peers;
}

// per-block sums of tiles[] in visible-set order
// The grid also zeroes the per-tile pair totals (T words) that the emission
// blocks add to.
__global__ void __launch_bounds__(GS_BLOCK) k_tile_sums(const uint32_t* __restrict__ order,
                                                        const uint32_t* __restrict__ vis_count,
                                                        const uint32_t* __restrict__ tiles,
                                                        uint32_t* __restrict__ bsum, uint32_t* __restrict__ tcount,
                                                        uint32_t T) {
    __shared__ uint32_t scratch[4];
    for (uint32_t i = blockIdx.x * GS_BLOCK + threadIdx.x; i < T; i += gridDim.x * GS_BLOCK) tcount[i] = 0u;
    const uint32_t V = *vis_count;
    const uint32_t base = blockIdx.x * GS_TILE_ITEMS + threadIdx.x * GS_ITEMS;
    uint32_t s = 0;
    if (blockIdx.x * GS_TILE_ITEMS < V) {
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k)
            if (base + k < V) s += tiles[order[base + k]];
    }
    const uint32_t t = block_sum_u32(s, scratch);
    if (threadIdx.x == 0) bsum[blockIdx.x] = t;
}

// Exclusive offsets in visible-set order: pair_offset[id] and offs_r[rank],
// with offs_r[V] = M as a sentinel.  Each block adds up the per-block sums of
// k_tile_sums itself, those before it for its offset and all of them for M
// (no separate scan pass).  Also publishes the pair count and the
// overflow flag, and for every 2048-pair emission block m the rank that holds
// its first pair (bstart[m], m < nbs): the rank whose pairs [off, off + t)
// contain m * 2048 writes it, so each entry has one writer.  On overflow
// (M > capacity) no pair is emitted and pair_offset[id] = 0xFFFFFFFF, so the
// per-primitive backward finds none of its slots in the buffer.
__global__ void __launch_bounds__(GS_BLOCK) k_offsets(
    const uint32_t* __restrict__ order, const uint32_t* __restrict__ vis_count, const uint32_t* __restrict__ tiles,
    const uint32_t* __restrict__ bsum, uint32_t capacity,
    uint32_t* __restrict__ pair_offset, uint32_t* __restrict__ offs_r, uint32_t* __restrict__ sort_count,
    uint32_t* __restrict__ num_pairs, gs_device_status* __restrict__ status, uint32_t* __restrict__ bstart,
    uint32_t nbs) {
    __shared__ uint32_t scratch[4];
    const uint32_t V = *vis_count;
    const uint32_t nbv = (V + GS_TILE_ITEMS - 1) / GS_TILE_ITEMS;     // blocks that hold visible ranks
    if (blockIdx.x > 0 && blockIdx.x >= nbv) return;
    uint32_t before;
    const uint32_t M = block_sum_prefix2(bsum, min(blockIdx.x, nbv), nbv, scratch, &before);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *num_pairs = M;
        *sort_count = M <= capacity ? M : 0u;
        offs_r[V] = M;
        if (M > capacity && status) {
            atomicOr(&status->flags, GS_DEV_PAIR_OVERFLOW);
            atomicMax(&status->required, M);
        }
    }
    if (blockIdx.x * GS_TILE_ITEMS >= V) return;
    const uint32_t base = blockIdx.x * GS_TILE_ITEMS + threadIdx.x * GS_ITEMS;
    uint32_t t[GS_ITEMS], g[GS_ITEMS];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < GS_ITEMS; ++k) {
        g[k] = (base + k < V) ? order[base + k] : 0u;
        t[k] = (base + k < V) ? tiles[g[k]] : 0u;
        s += t[k];
    }
    uint32_t tot;
    uint32_t off = block_excl_scan(s, scratch, &tot) + before;
#pragma unroll
    for (int k = 0; k < GS_ITEMS; ++k) {
        if (base + k >= V) break;
        pair_offset[g[k]] = M <= capacity ? off : 0xFFFFFFFFu;
        offs_r[base + k] = off;
        const uint64_t end = (uint64_t)off + t[k];
        for (uint64_t m = ((uint64_t)off + GS_TILE_ITEMS - 1) / GS_TILE_ITEMS; m < nbs && m * GS_TILE_ITEMS < end; ++m)
            bstart[m] = base + k;
        off += t[k];
    }
}

// Tiles up to which a block clears and reads the counters of all of them instead of
// finding the range its pairs span.  The range costs about 1 us in each of the two
// kernels (2170 tiles, pool in given order: emission and placement 31 us, with it 33)
// and saves passes over counters that stay 0 (32,400 tiles: 112 -> 78 us; 8160: 46 -> 44).
constexpr uint32_t kAllTiles = 4096;

// First and last tile of the block's keys (0xFFFFFFFF: no pair; a block holds at
// least one), within [0, T); all T tiles if there are few.  s: two words per wave.
// Every thread of the block must call it: it ends with a barrier.
__device__ __forceinline__ void block_key_range(const uint32_t (&key)[GS_ITEMS], uint32_t T, uint32_t* s, uint32_t* lo,
                                                uint32_t* up) {
    constexpr int kWaves = GS_BLOCK / GS_WAVE;
    if (T <= kAllTiles) {
        *lo = 0u;
        *up = T - 1u;
        __syncthreads();
        return;
    }
    uint32_t a = 0xFFFFFFFFu, b = 0u;
#pragma unroll
    for (int k = 0; k < GS_ITEMS; ++k) {
        a = min(a, key[k]);
        b = max(b, key[k] == 0xFFFFFFFFu ? 0u : key[k]);
    }
#pragma unroll
    for (int d = GS_WAVE / 2; d >= 1; d >>= 1) {
        a = min(a, (uint32_t)__shfl_xor((int)a, d, GS_WAVE));
        b = max(b, (uint32_t)__shfl_xor((int)b, d, GS_WAVE));
    }
    if (lane_id() == 0) {
        s[threadIdx.x / GS_WAVE] = a;
        s[kWaves + threadIdx.x / GS_WAVE] = b;
    }
    __syncthreads();
    *lo = min(min(s[0], s[1]), min(s[2], s[3]));
    *up = min(max(max(s[kWaves], s[kWaves + 1]), max(s[kWaves + 2], s[kWaves + 3])), T - 1u);
}

// Clears the nc counters of h (16-byte aligned).
__device__ __forceinline__ void clear_counts(uint32_t* h, uint32_t nc) {
    uint4* h4 = reinterpret_cast<uint4*>(h);
    for (uint32_t d = threadIdx.x; d < (nc + 3u) / 4u; d += GS_BLOCK) h4[d] = make_uint4(0u, 0u, 0u, 0u);
}

// Pair i belongs to the rank r with offs_r[r] <= i < offs_r[r+1] and covers tile
// number i - offs_r[r] of that primitive's rectangle (row-major).  A block takes 2048
// pairs, a thread eight in a row.  Every rank with a pair in the block leaves its id,
// rectangle and depth in LDS at its first pair's place; the last such place up to a
// thread's first pair (a running maximum over the block) names that pair's rank, and
// from there on the thread steps through the rectangles, taking up the next rank where
// it meets one: one division a thread and no search.  Tile (pkeys), primitive (pvals)
// and depth bits (pdepth) leave in 16-byte stores.  Then the block counts its pairs per
// tile in LDS (the same memory reused) and adds every non-zero count to the tile's total.
//
// What bounds it is the latency of a lone wave per SIMD and of the loads before it: a
// binary search over the ranks and a division for every pair took 6.4 of the 9.3 us of
// a block of 300 ranks.  Measured: 65k pairs on 256 tiles 12.4 -> 7.2 us, a 1M-primitive
// 1080p room's view 19.8 -> 14.0, 2.9M pairs at 3840x2160 28.4 -> 25.0.
__global__ void __launch_bounds__(GS_BLOCK) k_emit_pairs(
    const uint32_t* __restrict__ order, const uint32_t* __restrict__ vis_count, const uint32_t* __restrict__ offs_r,
    const uint32_t* __restrict__ bstart, const ushort4* __restrict__ rect, const float* __restrict__ depth,
    const uint32_t* __restrict__ sort_count, int32_t tiles_x, uint32_t T, uint32_t* __restrict__ pkeys,
    uint32_t* __restrict__ pvals, uint32_t* __restrict__ pdepth, uint32_t* __restrict__ tcount) {
    constexpr int kWaves = GS_BLOCK / GS_WAVE, kRounds = 4;
    constexpr uint32_t kNone = 0xFFFFFFFFu;     // no rank starts here (an id is below 2^31)
    static_assert(GS_ITEMS == 8, "a thread's pairs are two 16-byte words of each array");
    static_assert(GS_TILE_ITEMS * 16 >= kTileChunk * 4, "the tile histogram fits in the staging memory");
    __shared__ __align__(16) unsigned char s_mem[GS_TILE_ITEMS * 16];
    ushort4* s_rect = reinterpret_cast<ushort4*>(s_mem);
    uint32_t* s_gid = reinterpret_cast<uint32_t*>(s_mem + GS_TILE_ITEMS * 8);
    uint32_t* s_dep = reinterpret_cast<uint32_t*>(s_mem + GS_TILE_ITEMS * 12);
    __shared__ uint32_t s_key[2 * kWaves];
    __shared__ int s_last[kWaves];
    const uint32_t M = *sort_count;
    const uint32_t base = blockIdx.x * GS_TILE_ITEMS;
    if (base >= M) return;
    const uint32_t hi = min(base + (uint32_t)GS_TILE_ITEMS, M);
    // The ranks of the block's first and last pairs: the first from the table
    // k_offsets wrote; the next block's first rank bounds the last (it may start at
    // hi or share its offset with ranks without pairs), the last rank of all for the
    // last block.  They are at most GS_TILE_ITEMS + 1 when every rank holds >= 1 pair
    // (the visible set of gs_project's tile counts); a caller list with zero-tile ids
    // can span more, and then every pair's rank is searched for in global memory
    // instead (the last one whose offset is <= i: a zero-tile rank shares its
    // successor's offset), which grows with the logarithm of the ranks only.
    const uint32_t r0 = bstart[blockIdx.x];
    const uint32_t r1 = hi == M ? *vis_count - 1u : bstart[blockIdx.x + 1];
    const uint32_t nr = r1 - r0 + 1;
    const uint32_t skipped = base - offs_r[r0];       // pairs of the first rank before the block
    const uint32_t p0 = threadIdx.x * GS_ITEMS, i0 = base + p0;
    uint32_t gid[GS_ITEMS], dep[GS_ITEMS], key[GS_ITEMS];
    if (nr <= GS_TILE_ITEMS + 1) {
        uint4* own_gid = reinterpret_cast<uint4*>(s_gid + p0);
        own_gid[0] = own_gid[1] = make_uint4(kNone, kNone, kNone, kNone);
        __syncthreads();
        for (uint32_t j0 = threadIdx.x; j0 < nr; j0 += kRounds * GS_BLOCK) {
            // the ids of four rounds in flight together, then their rectangles and depths
            uint32_t g[kRounds], place[kRounds];
            ushort4 rc[kRounds];
            uint32_t dep[kRounds];
#pragma unroll
            for (int k = 0; k < kRounds; ++k) {
                const uint32_t j = j0 + k * GS_BLOCK;
                place[k] = kNone;
                if (j >= nr) continue;
                g[k] = order[r0 + j];
                const uint32_t off = offs_r[r0 + j];
                if (offs_r[r0 + j + 1] > off && off < hi) place[k] = j == 0u ? 0u : off - base;
            }
#pragma unroll
            for (int k = 0; k < kRounds; ++k) {
                if (place[k] == kNone) continue;
                rc[k] = rect[g[k]];
                dep[k] = __float_as_uint(depth[g[k]]);
            }
#pragma unroll
            for (int k = 0; k < kRounds; ++k) {
                if (place[k] == kNone) continue;
                s_gid[place[k]] = g[k];
                s_rect[place[k]] = rc[k];
                s_dep[place[k]] = dep[k];
            }
        }
        __syncthreads();
        ushort4 rc[GS_ITEMS];
        __builtin_memcpy(gid, __builtin_assume_aligned(s_gid + p0, 16), sizeof(gid));
        __builtin_memcpy(dep, __builtin_assume_aligned(s_dep + p0, 16), sizeof(dep));
        __builtin_memcpy(rc, __builtin_assume_aligned(s_rect + p0, 16), sizeof(rc));
        int last = -1;                              // the thread's last place that a rank starts at
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k) last = gid[k] != kNone ? (int)p0 + k : last;
        const int lane = lane_id(), wv = threadIdx.x / GS_WAVE;
        int upto = last;                            // the same over the wave's lanes up to this one
#pragma unroll
        for (int d = 1; d < GS_WAVE; d <<= 1) {
            const int o = __shfl_up(upto, d, GS_WAVE);
            upto = lane >= d ? max(upto, o) : upto;
        }
        if (lane == GS_WAVE - 1) s_last[wv] = upto;
        int at = __shfl_up(upto, 1, GS_WAVE);
        if (lane == 0) at = -1;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kWaves; ++i) at = i < wv ? max(at, s_last[i]) : at;
        // the rank of the thread's first pair, and that pair's place in its rectangle
        uint32_t g = gid[0], dp = dep[0];
        ushort4 r = rc[0];
        uint32_t local = threadIdx.x == 0 ? skipped : 0u;
        if (gid[0] == kNone) {                      // (place 0 always holds a rank)
            g = s_gid[at];
            dp = s_dep[at];
            r = s_rect[at];
            local = p0 - (uint32_t)at + (at == 0 ? skipped : 0u);
        }
        const uint32_t width = (uint32_t)(r.z - r.x);
        uint32_t row = local / width;
        uint32_t tx = r.x + (local - row * width), line = (r.y + row) * (uint32_t)tiles_x;
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k) {
            if (k > 0) {
                const bool next = gid[k] != kNone;
                const bool wrap = ++tx >= r.z;
                g = next ? gid[k] : g;
                dp = next ? dep[k] : dp;
                line = next ? rc[k].y * (uint32_t)tiles_x : (wrap ? line + (uint32_t)tiles_x : line);
                r.x = next ? rc[k].x : r.x;
                r.z = next ? rc[k].z : r.z;
                tx = next || wrap ? r.x : tx;
            }
            gid[k] = g;
            dep[k] = dp;
            key[k] = i0 + k < hi ? line + tx : 0xFFFFFFFFu;
        }
    } else {
        for (int k = 0; k < GS_ITEMS; ++k) {
            const uint32_t i = i0 + k;
            gid[k] = dep[k] = 0u;
            key[k] = 0xFFFFFFFFu;
            if (i >= hi) continue;
            uint32_t lo = r0, up = r0 + nr;
            while (up - lo > 1) {
                const uint32_t mid = (lo + up) >> 1;
                if (offs_r[mid] <= i) lo = mid; else up = mid;
            }
            gid[k] = order[lo];
            const ushort4 r = rect[gid[k]];
            const uint32_t local = i - offs_r[lo], width = (uint32_t)(r.z - r.x), row = local / width;
            key[k] = (r.y + row) * (uint32_t)tiles_x + r.x + (local - row * width);
            dep[k] = __float_as_uint(depth[gid[k]]);
        }
    }
    if (i0 + GS_ITEMS <= hi) {
        __builtin_memcpy(__builtin_assume_aligned(pkeys + i0, 16), key, sizeof(key));
        __builtin_memcpy(__builtin_assume_aligned(pvals + i0, 16), gid, sizeof(gid));
        __builtin_memcpy(__builtin_assume_aligned(pdepth + i0, 16), dep, sizeof(dep));
    } else {
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k) {
            if (i0 + k >= hi) break;
            pkeys[i0 + k] = key[k];
            pvals[i0 + k] = gid[k];
            pdepth[i0 + k] = dep[k];
        }
    }
    // counts per tile, over the tiles from the block's first to its last: in a
    // spatially ordered pool a block's pairs span a few rows of tiles
    uint32_t* h = reinterpret_cast<uint32_t*>(s_mem);
    uint32_t lo, up;
    block_key_range(key, T, s_key, &lo, &up);     // (the staging memory is free behind its barrier)
    for (uint32_t c0 = lo; c0 <= up; c0 += kTileChunk) {
        const uint32_t nc = min(kTileChunk, up - c0 + 1u);
        clear_counts(h, nc);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k)
            if (key[k] - c0 < nc) atomicAdd(&h[key[k] - c0], 1u);
        __syncthreads();
        for (uint32_t d = threadIdx.x; d < nc; d += GS_BLOCK) {
            const uint32_t c = h[d];
            if (c) atomicAdd(&tcount[c0 + d], c);
        }
        __syncthreads();    // before the next chunk clears the counters
    }
}

// Dispatch key of a tile from its pair count: an 8-bit code that never
// decreases with the count (exact below 16, then 16 steps per octave; counts
// of 2^19 and more share the top code), inverted so that ascending keys put
// the longest tiles first.
__device__ __forceinline__ uint32_t tile_order_key(uint32_t n) {
    uint32_t code = n;
    if (n >= 16u) {
        const uint32_t e = 31u - (uint32_t)__clz(n);      // >= 4
        code = e > 18u ? 255u : 16u * (e - 3u) + ((n >> (e - 4u)) & 15u);
    }
    return 255u - code;
}

// Tiles with fewer pairs than this are depth-sorted by one wave in registers;
// the order key is monotone in the count, so these are exactly the tiles with
// keys above long_key, and the dispatch order puts all others first.  Where the tiles
// leave most of the chip idle (FEW, at most two per compute unit) a tile's own time
// counts: its waves share it from 256 pairs on, with as few keys a lane as hold it
// (256 tiles with one of 598 pairs: 15.8 -> 11.7 us).  With many tiles the longer code
// and the barriers cost more (8160 tiles of a 1M room: 30 -> 35 us).  In between it is
// the pairs a tile that decide, not known to the host.  Measured on a ring of 20k, 60k
// and 150k primitives (65k, 137k and 270k pairs on 475 tiles, 273k, 467k and 762k on
// 3600), the other form -> FEW: 475 tiles 18.4 -> 12.2, 22.7 -> 23.3, 108 -> 108 us; 578
// tiles 18.2 -> 11.1, 21.6 -> 22.1, 82.5 -> 82.1; 1900 tiles 16.6 -> 10.6, 19.0 -> 20.4,
// 24.9 -> 25.4; 3600 tiles 16.0 -> 9.9, 19.5 -> 15.4, 28.3 -> 25.6.  The line is at the
// lower end, below which the chip has idle units whatever the tiles hold; up to a few
// thousand tiles FEW would mostly gain too, and lost 7% at worst here.
template <bool FEW>
constexpr uint32_t kWaveSortMax = FEW ? 256u : 512u;
template <bool FEW>
constexpr uint32_t kLongKey = FEW ? 255u - 80u : 255u - 96u;   // tile_order_key: code 16 * (8 - 3), 16 * (9 - 3)

// Exclusive scan over the 4 waves of a workgroup of GS_BLOCK threads is
// block_excl_scan.

// Tiles per workgroup of the finishing grid (2 per thread), and the totals
// each thread loads per pass over all tiles (one pass up to 8192 tiles).
constexpr uint32_t kFinishPer = 2;
constexpr uint32_t kFinishSeg = kFinishPer * GS_BLOCK;
constexpr int kFinishLoads = 32;

// From the per-tile totals: the tile ranges (exclusive scan in tile order;
// [0, 0) for a tile without pairs), the placement cursors (each range's
// start), the dispatch order (tiles by ascending tile_order_key, equal keys
// by ascending id) with one record per dispatch position (tile, range start,
// pair count), and the number of tiles with keys up to long_key, which
// the order puts first.  Workgroup b owns the tiles [b*kFinishSeg, ..) of one
// segment.  It reads every total (all loads of a pass in flight together):
// their sum before the segment starts its ranges, and the key counts over all
// tiles and over the tiles before the segment give each key's first position
// for the segment; the segment's own totals and range starts stay in LDS.
// Inside the segment, wave w owns a contiguous quarter: it counts its keys,
// the counts give every (wave, key) its first position, and the wave then
// places its tiles 64 at a time, each lane ranked among the earlier lanes
// with its key.
__global__ void __launch_bounds__(GS_BLOCK) k_tile_finish(const uint32_t* __restrict__ tcount, uint32_t T,
                                                          uint32_t* __restrict__ ranges,
                                                          uint32_t* __restrict__ cursor,
                                                          uint32_t* __restrict__ order, uint4* __restrict__ rec,
                                                          uint32_t long_key, uint32_t* __restrict__ n_long) {
    constexpr int kWaves = GS_BLOCK / GS_WAVE;
    __shared__ uint32_t s_all[256], s_before[256];
    __shared__ uint32_t s_wc[kWaves][256];
    __shared__ uint32_t s_cnt[kFinishSeg], s_sta[kFinishSeg];
    __shared__ uint32_t scratch[4];
    const uint32_t tid = threadIdx.x;
    const uint32_t w = tid / GS_WAVE;
    const uint32_t lane = lane_id();
    const uint32_t lo = blockIdx.x * kFinishSeg, hi = min(lo + kFinishSeg, T);
    s_all[tid] = 0u;
    s_before[tid] = 0u;
    s_wc[0][tid] = 0u; s_wc[1][tid] = 0u; s_wc[2][tid] = 0u; s_wc[3][tid] = 0u;
    __syncthreads();
    // every total: key counts over all tiles and before the segment, the pairs
    // before it; the segment's totals to LDS
    uint32_t before = 0;
    for (uint32_t r0 = 0; r0 < T; r0 += GS_BLOCK * kFinishLoads) {
        uint32_t c[kFinishLoads];
#pragma unroll
        for (int k = 0; k < kFinishLoads; ++k) c[k] = tcount[min(r0 + k * GS_BLOCK + tid, T - 1u)];
#pragma unroll
        for (int k = 0; k < kFinishLoads; ++k) loaded(c[k]);
#pragma unroll
        for (int k = 0; k < kFinishLoads; ++k) {
            const uint32_t t = r0 + k * GS_BLOCK + tid;
            if (t < T) {
                const uint32_t key = tile_order_key(c[k]);
                atomicAdd(&s_all[key], 1u);
                if (t < lo) {
                    atomicAdd(&s_before[key], 1u);
                    before += c[k];
                } else if (t < hi) {
                    s_cnt[t - lo] = c[k];
                }
            }
        }
    }
    __syncthreads();
    // the segment: kFinishPer consecutive tiles per thread
    const uint32_t l0 = tid * kFinishPer;
    uint32_t c[kFinishPer], csum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kFinishPer; ++k) {
        c[k] = lo + l0 + k < hi ? s_cnt[l0 + k] : 0u;
        csum += c[k];
    }
    uint32_t tot;
    const uint32_t pre = block_sum_u32(before, scratch);       // (the block's sum of `before`)
    uint32_t run = block_excl_scan(csum, scratch, &tot) + pre;
#pragma unroll
    for (uint32_t k = 0; k < kFinishPer; ++k) {
        const uint32_t t = lo + l0 + k;
        if (t < hi) {
            ranges[2 * t] = c[k] ? run : 0u;
            ranges[2 * t + 1] = c[k] ? run + c[k] : 0u;
            cursor[t] = run;
            s_sta[l0 + k] = c[k] ? run : 0u;
        }
        run += c[k];
    }
    // key d (thread d): its first position for the segment
    {
        uint32_t ktot;
        const uint32_t kstart = block_excl_scan(s_all[tid], scratch, &ktot);
        if (blockIdx.x == 0 && tid == long_key + 1u) *n_long = kstart;   // tiles with key <= long_key come first
        s_all[tid] = kstart + s_before[tid];
    }
    // per wave: key counts of its quarter of the segment (its lanes' tiles, in order)
    const uint32_t qlo = w * (kFinishSeg / kWaves);                         // segment-relative
    const uint32_t qhi = min(qlo + kFinishSeg / kWaves, hi - lo);
    uint32_t* wc = s_wc[w];
    __syncthreads();
    for (uint32_t l = qlo + lane; l < qhi; l += GS_WAVE) atomicAdd(&wc[tile_order_key(s_cnt[l])], 1u);
    __syncthreads();
    {
        uint32_t b = s_all[tid];
        const uint32_t c0 = s_wc[0][tid], c1 = s_wc[1][tid], c2 = s_wc[2][tid];
        s_wc[0][tid] = b;
        s_wc[1][tid] = b + c0;
        s_wc[2][tid] = b + c0 + c1;
        s_wc[3][tid] = b + c0 + c1 + c2;
    }
    __syncthreads();
    // placement: the quarter's tiles 64 at a time
    const uint64_t lt = lanemask_lt();
    for (uint32_t b0 = qlo; b0 < qhi; b0 += GS_WAVE) {
        const uint32_t l = b0 + lane;
        const bool valid = l < qhi;
        const uint32_t cnt = valid ? s_cnt[l] : 0u;
        const uint32_t sta = valid ? s_sta[l] : 0u;
        const uint32_t key = tile_order_key(cnt);
        const uint64_t peers = match_digit(key, valid, 8);
        const uint32_t bw = valid ? wc[key] : 0u;
        if (valid) {
            const uint32_t pos = bw + (uint32_t)popc64(peers & lt);
            order[pos] = lo + l;
            rec[pos] = make_uint4(lo + l, sta, cnt, 0u);
        }
        // all reads of this round precede the leaders' updates
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (valid && (peers & lt) == 0ull) wc[key] = bw + (uint32_t)popc64(peers);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// A pair's record: 12 bytes without padding (16 cost the sort 1 to 2 us a view in
// cache misses).
struct PairRec {
    uint32_t emit, depth, gid;
};
static_assert(sizeof(PairRec) == 12, "three words a pair in the workspace");

// The 64-bit key of a record, and a key in its place (the primitive stays).
__device__ __forceinline__ unsigned long long rec_key(const PairRec& r) {
    return ((unsigned long long)r.depth << 32) | r.emit;
}
__device__ __forceinline__ void put_key(PairRec* r, unsigned long long k) {
    r->emit = (uint32_t)k;
    r->depth = (uint32_t)(k >> 32);
}

// Placement of the emitted pairs in their tiles' ranges: the block ranks its
// pairs per tile in LDS, claims one run of slots per distinct tile from the
// tile's cursor, and writes each pair's record at its slot: the depth-sort key (the
// depth bits above the emission position) and the primitive.  What bounds it are the
// scattered stores, by their number more than their bytes: one of 12 bytes a pair in
// place of 8 + 4 in two arrays.  Measured: 2.9M pairs at 3840x2160 51.7 -> 36.9 us (with
// the sort that reads them 95.4 -> 80.3), a 1M-primitive room's view 25.0 -> 21.1 (53.3 ->
// 50.8).  The key alone, with the primitive looked up by emission position, placed 4 us
// faster still and cost the sort 17.
__global__ void __launch_bounds__(GS_BLOCK) k_tile_scatter(const uint32_t* __restrict__ pkeys,
                                                           const uint32_t* __restrict__ pvals,
                                                           const uint32_t* __restrict__ pdepth,
                                                           const uint32_t* __restrict__ sort_count, uint32_t T,
                                                           uint32_t* __restrict__ cursor,
                                                           PairRec* __restrict__ rec) {
    __shared__ __align__(16) uint32_t h[kTileChunk];
    __shared__ uint32_t s_key[2 * GS_BLOCK / GS_WAVE];
    const uint32_t M = *sort_count;
    const uint32_t base = blockIdx.x * GS_TILE_ITEMS + threadIdx.x;
    if (blockIdx.x * GS_TILE_ITEMS >= M) return;
    uint32_t key[GS_ITEMS], dep[GS_ITEMS], gid[GS_ITEMS], rk[GS_ITEMS];
#pragma unroll
    for (int k = 0; k < GS_ITEMS; ++k) {
        const uint32_t i = base + k * GS_BLOCK;
        key[k] = i < M ? pkeys[i] : 0xFFFFFFFFu;
        dep[k] = i < M ? pdepth[i] : 0u;
        gid[k] = i < M ? pvals[i] : 0u;
        rk[k] = 0u;
    }
    uint32_t lo, up;
    block_key_range(key, T, s_key, &lo, &up);
    for (uint32_t c0 = lo; c0 <= up; c0 += kTileChunk) {
        const uint32_t nc = min(kTileChunk, up - c0 + 1u);
        clear_counts(h, nc);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k)
            if (key[k] - c0 < nc) rk[k] = atomicAdd(&h[key[k] - c0], 1u);
        __syncthreads();
        for (uint32_t d = threadIdx.x; d < nc; d += GS_BLOCK) {
            const uint32_t c = h[d];
            if (c) h[d] = atomicAdd(&cursor[c0 + d], c);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k)
            if (key[k] - c0 < nc) {
                const uint32_t at = h[key[k] - c0] + rk[k];
                rec[at] = PairRec{base + k * GS_BLOCK, dep[k], gid[k]};
            }
        __syncthreads();    // before the next chunk clears the counters
    }
}

// Per-tile ordering.  A tile's pairs arrive in its range in any order, each
// as a 64-bit key (depth bits above the emission position) and the pair's
// primitive.  The fast paths sort the 32-bit depth bits alone, each with the
// index of its slot as payload; pairs with equal depth bits (a run of
// neighbours in that order) are then placed by their emission positions,
// which gives the order by (depth bits, emission position).  A tile with a
// run longer than kRunMax (or a depth key equal to the padding value) is
// sorted again, exactly, on the 64-bit keys.
constexpr unsigned long long kKeyMax = ~0ull;
constexpr uint32_t kDepthPad = 0xFFFFFFFFu;
constexpr uint32_t kRunMax = 64;

// Bitonic network, in the variant whose compare-exchanges all put the smaller
// key at the lower index: each merge of width k (a power of two) first
// compares i with its mirror i ^ (k - 1), then i with i ^ j for j = k/4 .. 1.

// The exact network on a segment of global memory of any length n, by a
// whole workgroup: entries at n and beyond are taken as kKeyMax, so a
// compare-exchange that reaches past the data leaves the lower (real) entry
// in place.  Only the keys move.
__device__ void bitonic_global(PairRec* s, uint32_t n) {
    uint32_t np = 1;
    while (np < n) np <<= 1;
    for (uint32_t k = 2; k <= np; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            const uint32_t mask = (j == (k >> 1)) ? (k - 1) : j;
            for (uint32_t c = threadIdx.x; c < (np >> 1); c += GS_BLOCK) {
                const uint32_t i = ((c & ~(j - 1)) << 1) | (c & (j - 1));
                const uint32_t q = i ^ mask;
                if (q >= n) continue;
                const unsigned long long a = rec_key(s[i]), b = rec_key(s[q]);
                if (b < a) {
                    put_key(&s[i], b);
                    put_key(&s[q], a);
                }
            }
            __threadfence_block();
            __syncthreads();
        }
    }
}

// LDS accesses of one wave, ordered (no other wave touches the memory).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Writes sorted pair `at` of tile t: its emission position, primitive id (pvals holds
// them by emission position) and optional 64-bit key.
__device__ __forceinline__ void put_sorted(uint32_t t, uint32_t at, unsigned long long k,
                                           const uint32_t* __restrict__ pvals, uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                                           uint64_t* __restrict__ keys64) {
    vals[at] = pvals[(uint32_t)k];
    pair_emit[at] = (uint32_t)k;
    if (keys64) keys64[at] = ((uint64_t)t << 32) | (k >> 32);
}

// The exact network over the n (<= 512) 64-bit keys of a tile by one wave,
// in the wave's own LDS (sk: 512 entries).
__device__ void wave_sort_tile64(uint32_t t, uint32_t start, uint32_t n, const PairRec* __restrict__ skey,
                                 const uint32_t* __restrict__ pvals, unsigned long long* sk,
                                 uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                                 uint64_t* __restrict__ keys64) {
    const uint32_t lane = lane_id();
    uint32_t np = 2;
    while (np < n) np <<= 1;
    for (uint32_t i = lane; i < np; i += GS_WAVE) {
        sk[i] = i < n ? rec_key(skey[start + i]) : kKeyMax;
    }
    wave_sync();
    for (uint32_t k = 2; k <= np; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            const uint32_t mask = (j == (k >> 1)) ? (k - 1) : j;
            for (uint32_t c = lane; c < (np >> 1); c += GS_WAVE) {
                const uint32_t i = ((c & ~(j - 1)) << 1) | (c & (j - 1));
                const uint32_t q = i ^ mask;
                const unsigned long long a = sk[i], b = sk[q];
                if (b < a) {
                    sk[i] = b;
                    sk[q] = a;
                }
            }
            wave_sync();
        }
    }
    for (uint32_t i = lane; i < n; i += GS_WAVE) put_sorted(t, start + i, sk[i], pvals, pair_emit, vals, keys64);
    wave_sync();
}

// Lane l's value of lane l ^ M: DPP inside rows for the masks 1, 2, 3, 7 and
// 15, a swizzle inside 32-lane halves for the other masks below 32, a
// permute for 32 and 63.  Every lane of the wave must be active.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    if constexpr (M == 1)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);    // quad_perm 1,0,3,2
    else if constexpr (M == 2)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);    // quad_perm 2,3,0,1
    else if constexpr (M == 3)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x1B, 0xF, 0xF, false);    // quad_perm 3,2,1,0
    else if constexpr (M == 7)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    else if constexpr (M == 15)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false);   // row_mirror
    else if constexpr (M < 32)
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (M << 10) | 0x1F);            // and 31, xor M
    else
        return __shfl_xor(v, M, GS_WAVE);
}

// Compare-exchange inside a lane: the smaller key (and its payload) to a.
__device__ __forceinline__ void cmpx32(uint32_t& a, uint32_t& pa, uint32_t& b, uint32_t& pb) {
    const bool sw = b < a;
    const uint32_t lo = sw ? b : a, hi = sw ? a : b, plo = sw ? pb : pa, phi = sw ? pa : pb;
    a = lo;
    b = hi;
    pa = plo;
    pb = phi;
}

// One side of a step across lanes or waves: the lower side keeps the
// smaller key, the upper side the larger.
__device__ __forceinline__ void keep32(uint32_t& v, uint32_t& p, uint32_t o, uint32_t op, bool lower) {
    const bool take = lower ? (o < v) : (v < o);
    v = take ? o : v;
    p = take ? op : p;
}

// The network on the 64 K keys of one wave in registers: element i = lane * K
// + r sits in register r of its lane, so a step at distance below K stays
// inside a lane and one at a larger distance pairs lane l with lane l ^
// (distance / K), same register.

// Steps i against i ^ j for j = J, J/2, .. 1.
template <int K, int J>
__device__ __forceinline__ void tail32(uint32_t (&v)[K], uint32_t (&p)[K], uint32_t lane) {
    if constexpr (J > 0) {
        if constexpr (J < K) {
#pragma unroll
            for (int r = 0; r < K; ++r)
                if ((r & J) == 0) cmpx32(v[r], p[r], v[r | J], p[r | J]);
        } else {
            const bool lower = (lane & (uint32_t)(J / K)) == 0;
#pragma unroll
            for (int r = 0; r < K; ++r) keep32(v[r], p[r], lane_xor<J / K>(v[r]), lane_xor<J / K>(p[r]), lower);
        }
        tail32<K, J / 2>(v, p, lane);
    }
}

// Mirror step of a merge of width KK: i against i ^ (KK - 1).
template <int K, int KK>
__device__ __forceinline__ void mirror32(uint32_t (&v)[K], uint32_t (&p)[K], uint32_t lane) {
    if constexpr (KK <= K) {
#pragma unroll
        for (int r = 0; r < K; ++r)
            if ((r & (KK / 2)) == 0) cmpx32(v[r], p[r], v[r ^ (KK - 1)], p[r ^ (KK - 1)]);
    } else {
        const bool lower = (lane & (uint32_t)(KK / K / 2)) == 0;
        uint32_t o[K], op[K];
#pragma unroll
        for (int r = 0; r < K; ++r) {
            o[r] = lane_xor<KK / K - 1>(v[r ^ (K - 1)]);
            op[r] = lane_xor<KK / K - 1>(p[r ^ (K - 1)]);
        }
#pragma unroll
        for (int r = 0; r < K; ++r) keep32(v[r], p[r], o[r], op[r], lower);
    }
}

// Merges of width 2 .. KK: every block of KK elements ascending.
template <int K, int KK>
__device__ __forceinline__ void net32(uint32_t (&v)[K], uint32_t (&p)[K], uint32_t lane) {
    if constexpr (KK >= 2) {
        net32<K, KK / 2>(v, p, lane);
        mirror32<K, KK>(v, p, lane);
        tail32<K, KK / 4>(v, p, lane);
    }
}

// Depth bits and emission position of the key of record i (its high and low words).
__device__ __forceinline__ uint32_t key_depth(const PairRec* __restrict__ skey, uint32_t i) {
    return skey[i].depth;
}
__device__ __forceinline__ uint32_t key_emit(const PairRec* __restrict__ skey, uint32_t i) {
    return skey[i].emit;
}

// Writes the pairs of a tile sorted by depth bits: sorted pair i is slot p.
__device__ __forceinline__ void put_by_slot(uint32_t t, uint32_t start, uint32_t i, uint32_t depth, uint32_t p,
                                            const PairRec* __restrict__ skey,
                                            uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                                            uint64_t* __restrict__ keys64) {
    const PairRec r = skey[start + p];
    vals[start + i] = r.gid;
    pair_emit[start + i] = r.emit;
    if (keys64) keys64[start + i] = ((uint64_t)t << 32) | depth;
}

// Runs of equal depth bits.  sk[0..n) holds a tile's keys in the order of
// their depth bits (ties in any order).  long_run: some
// run is longer than kRunMax (then entry i and entry i - kRunMax share their
// depth bits).  place_runs writes sorted pair i for i = first, first + step,
// ..: an entry outside a run stays at i; one inside a run [a, b) goes to a +
// the number of the run's entries with a smaller key (emission position).
__device__ __forceinline__ uint32_t hi32(unsigned long long k) { return (uint32_t)(k >> 32); }

__device__ __forceinline__ bool long_run(const unsigned long long* sk, uint32_t n, uint32_t first, uint32_t step) {
    bool bad = false;
    for (uint32_t i = first + kRunMax; i < n; i += step) bad |= hi32(sk[i]) == hi32(sk[i - kRunMax]);
    return bad;
}

__device__ __forceinline__ void place_runs(uint32_t t, uint32_t start, uint32_t n, const unsigned long long* sk,
                                           const uint32_t* __restrict__ pvals, uint32_t first, uint32_t step,
                                           uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                                           uint64_t* __restrict__ keys64) {
    for (uint32_t i = first; i < n; i += step) {
        const unsigned long long k = sk[i];
        const uint32_t d = hi32(k);
        uint32_t a = i, b = i + 1;
        while (a > 0 && hi32(sk[a - 1]) == d) --a;
        while (b < n && hi32(sk[b]) == d) ++b;
        uint32_t at = a;
        for (uint32_t j = a; j < b; ++j) at += sk[j] < k ? 1u : 0u;
        put_sorted(t, start + at, k, pvals, pair_emit, vals, keys64);
    }
}

// One wave sorts the n (<= 64 K) pairs of one tile: the fast path in
// registers, else wave_sort_tile64 in the wave's LDS.
template <int K>
__device__ __forceinline__ void wave_sort_tile(uint32_t t, uint32_t start, uint32_t n,
                                               const PairRec* __restrict__ skey,
                                               const uint32_t* __restrict__ pvals, unsigned long long* sk,
                                               uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                                               uint64_t* __restrict__ keys64) {
    const uint32_t lane = lane_id();
    uint32_t v[K], p[K];
    bool odd = false;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        const uint32_t i = lane * K + r;
        v[r] = i < n ? key_depth(skey, start + i) : kDepthPad;
        p[r] = i;
        odd |= i < n && v[r] == kDepthPad;
    }
    bool tie = false;
    if (__ballot(odd) == 0ull) {
        net32<K, GS_WAVE * K>(v, p, lane);
        // equal neighbours in the sorted order: i and i + 1 < n
#pragma unroll
        for (int r = 0; r + 1 < K; ++r) tie |= lane * K + r + 1 < n && v[r] == v[r + 1];
        const uint32_t next = __shfl_down(v[0], 1, GS_WAVE);
        tie |= lane + 1 < GS_WAVE && (lane + 1) * K < n && v[K - 1] == next;
    }
    if (__ballot(odd) != 0ull) {
        wave_sort_tile64(t, start, n, skey, pvals, sk, pair_emit, vals, keys64);
        return;
    }
    if (__ballot(tie) == 0ull) {
#pragma unroll
        for (int r = 0; r < K; ++r)
            if (lane * K + r < n) put_by_slot(t, start, lane * K + r, v[r], p[r], skey, pair_emit, vals, keys64);
        return;
    }
    // equal depth bits: the sorted keys to LDS, then each run placed by emission position
#pragma unroll
    for (int r = 0; r < K; ++r) {
        const uint32_t i = lane * K + r;
        if (i < n) sk[i] = ((unsigned long long)v[r] << 32) | key_emit(skey, start + p[r]);
    }
    wave_sync();
    if (__ballot(long_run(sk, n, lane, GS_WAVE)) != 0ull) {
        wave_sync();
        wave_sort_tile64(t, start, n, skey, pvals, sk, pair_emit, vals, keys64);
        return;
    }
    place_runs(t, start, n, sk, pvals, lane, GS_WAVE, pair_emit, vals, keys64);
    wave_sync();
}

// Long tiles: kWaveSortMax<FEW> .. kLongCap pairs are sorted by the workgroup's
// waves in registers, 8 keys a lane (FEW: 2, 4 or 8); merges wider than one wave take
// their cross-wave steps through LDS.  Longer tiles take the exact network in
// global memory.
constexpr int kSortWaves = GS_BLOCK / GS_WAVE;
constexpr int kLongK = 8;                                // most keys per lane
constexpr uint32_t kLongCap = GS_BLOCK * kLongK;
// Workgroups per compute unit of the persistent depth-sort grid.
constexpr uint32_t kDepthSortBlocksPerCU = 8;

// The exact network over the n (<= kLongCap) 64-bit keys skey[start ..
// start + n) by the whole workgroup in LDS: sorted keys in sk[0..n).
__device__ void block_sort_lds64(uint32_t start, uint32_t n, const PairRec* __restrict__ skey,
                                 unsigned long long* sk) {
    uint32_t np = 2;
    while (np < n) np <<= 1;
    for (uint32_t i = threadIdx.x; i < np; i += GS_BLOCK) {
        sk[i] = i < n ? rec_key(skey[start + i]) : kKeyMax;
    }
    __syncthreads();
    for (uint32_t k = 2; k <= np; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            const uint32_t mask = (j == (k >> 1)) ? (k - 1) : j;
            for (uint32_t c = threadIdx.x; c < (np >> 1); c += GS_BLOCK) {
                const uint32_t i = ((c & ~(j - 1)) << 1) | (c & (j - 1));
                const uint32_t q = i ^ mask;
                const unsigned long long a = sk[i], b = sk[q];
                if (b < a) {
                    sk[i] = b;
                    sk[q] = a;
                }
            }
            __syncthreads();
        }
    }
}

// The exact network over the n (<= kLongCap) 64-bit keys of a tile by the
// whole workgroup in LDS, written out in order.
__device__ void block_sort_tile64(uint32_t t, uint32_t start, uint32_t n, const PairRec* __restrict__ skey,
                                  const uint32_t* __restrict__ pvals, unsigned long long* sk,
                                  uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                                  uint64_t* __restrict__ keys64) {
    block_sort_lds64(start, n, skey, sk);
    for (uint32_t i = threadIdx.x; i < n; i += GS_BLOCK) put_sorted(t, start + i, sk[i], pvals, pair_emit, vals, keys64);
    __syncthreads();
}

// Number of keys below each of the thread's R keys in the ascending keys
// sk[0..m) (keys are unique): a branch-free binary search, the R searches
// stepping together.
template <int R>
__device__ __forceinline__ void rank_in(const unsigned long long* sk, uint32_t m, const unsigned long long (&key)[R],
                                        uint32_t (&pos)[R]) {
    uint32_t step = 1;
    while (step <= m) step <<= 1;
#pragma unroll
    for (int k = 0; k < R; ++k) pos[k] = 0;
    for (step >>= 1; step > 0; step >>= 1) {
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (pos[k] + step <= m && sk[pos[k] + step - 1] < key[k]) pos[k] += step;
    }
}

// A tile of kLongCap < n <= 2 kLongCap pairs: its first kLongCap keys and the
// rest are each sorted exactly in LDS, and every key goes to its index in
// its own run plus its rank in the other run (the merged order; keys are
// unique).  Each sorted run is kept in its own place in global memory (this
// workgroup's segment) while the other one sits in LDS; the ranks are
// searched kRankGroup keys at a time per thread.
constexpr int kRankGroup = 4;

// The keys of run [r0, r0 + m) of the segment, ranked in the ascending keys
// sk[0..mo) in LDS; key i of the run goes to r_out + i + its rank.
__device__ __forceinline__ void place_ranked(uint32_t t, uint32_t start, uint32_t r0, uint32_t m, uint32_t r_out,
                                             const PairRec* __restrict__ skey,
                                             const uint32_t* __restrict__ pvals, const unsigned long long* sk,
                                             uint32_t mo, uint32_t* __restrict__ pair_emit,
                                             uint32_t* __restrict__ vals, uint64_t* __restrict__ keys64) {
    constexpr uint32_t kGroupSpan = kRankGroup * GS_BLOCK;
#pragma unroll 1
    for (uint32_t g = 0; g < m; g += kGroupSpan) {
        unsigned long long kk[kRankGroup];
        uint32_t rk[kRankGroup];
#pragma unroll
        for (int k = 0; k < kRankGroup; ++k) {
            const uint32_t i = min(g + threadIdx.x + k * GS_BLOCK, m - 1u);
            kk[k] = rec_key(skey[start + r0 + i]);
        }
        rank_in<kRankGroup>(sk, mo, kk, rk);
#pragma unroll
        for (int k = 0; k < kRankGroup; ++k) {
            const uint32_t i = g + threadIdx.x + k * GS_BLOCK;
            if (i < m) put_sorted(t, start + r_out + i + rk[k], kk[k], pvals, pair_emit, vals, keys64);
        }
    }
}

__device__ void sort_two_runs(uint32_t t, uint32_t start, uint32_t n, PairRec* __restrict__ skey,
                              const uint32_t* __restrict__ pvals, unsigned long long* sk,
                              uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                              uint64_t* __restrict__ keys64) {
    const uint32_t tid = threadIdx.x;
    const uint32_t na = kLongCap, nb = n - kLongCap;
    // the first run sorted, to its place
    block_sort_lds64(start, na, skey, sk);
    for (uint32_t i = tid; i < na; i += GS_BLOCK) put_key(&skey[start + i], sk[i]);
    __threadfence_block();
    __syncthreads();
    // the second run sorted (in LDS); the first run's keys placed by their ranks in it
    block_sort_lds64(start + na, nb, skey, sk);
    place_ranked(t, start, 0u, na, 0u, skey, pvals, sk, nb, pair_emit, vals, keys64);
    // the second run to its place, the first back to LDS; the second run's keys placed
    for (uint32_t i = tid; i < nb; i += GS_BLOCK) put_key(&skey[start + na + i], sk[i]);
    __threadfence_block();
    __syncthreads();
    for (uint32_t i = tid; i < na; i += GS_BLOCK) sk[i] = rec_key(skey[start + i]);
    __syncthreads();
    place_ranked(t, start, na, nb, 0u, skey, pvals, sk, na, pair_emit, vals, keys64);
    __syncthreads();
}

// A tile by the whole workgroup, exactly: up to 2 kLongCap pairs as two runs
// in LDS, longer ones in place in global memory.
__device__ void sort_huge_tile(uint32_t t, uint32_t start, uint32_t n, PairRec* __restrict__ skey,
                               const uint32_t* __restrict__ pvals, unsigned long long* sk,
                               uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                               uint64_t* __restrict__ keys64) {
    if (n <= 2 * kLongCap) {
        sort_two_runs(t, start, n, skey, pvals, sk, pair_emit, vals, keys64);
        return;
    }
    PairRec* key = skey + start;
    bitonic_global(key, n);
    for (uint32_t i = threadIdx.x; i < n; i += GS_BLOCK) put_sorted(t, start + i, rec_key(key[i]), pvals, pair_emit, vals, keys64);
}

// One cross-wave step of a long tile: element i (register r of lane l of
// wave w, i = (w * 64 + l) * K + r) against element i ^ mask.  Key and slot
// go through LDS as one word pair, r-major (address r * 256 + i / K), so the
// lanes of one access touch consecutive words.
template <int K>
__device__ __forceinline__ void long_exchange(uint32_t (&v)[K], uint32_t (&p)[K], bool act, uint32_t ibase,
                                              uint32_t mask, unsigned long long* s_kv) {
    constexpr uint32_t kStride = GS_BLOCK;
    const uint32_t hb = 1u << (31 - __clz(mask));          // the highest bit of mask decides the side
    if (act) {
#pragma unroll
        for (int r = 0; r < K; ++r) s_kv[r * kStride + (ibase / K)] = ((unsigned long long)p[r] << 32) | v[r];
    }
    __syncthreads();
    if (act) {
        const bool lower = (ibase & hb) == 0;              // hb >= 64 K > r: one side for all r
#pragma unroll
        for (int r = 0; r < K; ++r) {
            const uint32_t q = (ibase + r) ^ mask;
            const unsigned long long kv = s_kv[(q % K) * kStride + q / K];
            keep32(v[r], p[r], (uint32_t)kv, (uint32_t)(kv >> 32), lower);
        }
    }
    __syncthreads();
}

// A long tile (at most 256 K pairs) by the whole workgroup, K keys a lane.
template <int K>
__device__ __forceinline__ void sort_long_tile(uint32_t t, uint32_t start, uint32_t n, PairRec* __restrict__ skey,
                               const uint32_t* __restrict__ pvals, unsigned long long* s_kv,
                               uint32_t* s_first, uint32_t* __restrict__ pair_emit, uint32_t* __restrict__ vals,
                               uint64_t* __restrict__ keys64) {
    const uint32_t w = threadIdx.x / GS_WAVE, lane = lane_id();
    constexpr uint32_t kWave = GS_WAVE * K;      // keys of a wave
    uint32_t np = kWave;
    while (np < n) np <<= 1;
    const bool act = w < np / kWave;
    const uint32_t ibase = w * kWave + lane * K;
    uint32_t v[K], p[K];
    bool odd = false;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        const uint32_t i = ibase + r;
        v[r] = act && i < n ? key_depth(skey, start + i) : kDepthPad;
        p[r] = i;
        odd |= act && i < n && v[r] == kDepthPad;
    }
    if (__syncthreads_or(odd)) {
        block_sort_tile64(t, start, n, skey, pvals, s_kv, pair_emit, vals, keys64);
        return;
    }
    if (act) net32<K, (int)kWave>(v, p, lane);
    for (uint32_t kk = 2 * kWave; kk <= np; kk <<= 1) {
        long_exchange<K>(v, p, act, ibase, kk - 1, s_kv);
        for (uint32_t j = kk >> 2; j >= kWave; j >>= 1) long_exchange<K>(v, p, act, ibase, j, s_kv);
        if (act) tail32<K, (int)kWave / 2>(v, p, lane);
    }
    // equal neighbours: inside a lane, to the next lane, to the next wave
    if (act && lane == 0) s_first[w] = v[0];
    __syncthreads();
    bool tie = false;
    if (act) {
#pragma unroll
        for (int r = 0; r + 1 < K; ++r) tie |= ibase + r + 1 < n && v[r] == v[r + 1];
        const uint32_t next = __shfl_down(v[0], 1, GS_WAVE);
        if (lane + 1 < GS_WAVE)
            tie |= ibase + K < n && v[K - 1] == next;
        else if (w + 1 < np / kWave)
            tie |= ibase + K < n && v[K - 1] == s_first[w + 1];
    }
    if (!__syncthreads_or(tie)) {
        if (act) {
#pragma unroll
            for (int r = 0; r < K; ++r)
                if (ibase + r < n) put_by_slot(t, start, ibase + r, v[r], p[r], skey, pair_emit, vals, keys64);
        }
        return;
    }
    // equal depth bits: the sorted keys to LDS, then each run placed by emission position
    if (act) {
#pragma unroll
        for (int r = 0; r < K; ++r) {
            const uint32_t i = ibase + r;
            if (i < n) s_kv[i] = ((unsigned long long)v[r] << 32) | key_emit(skey, start + p[r]);
        }
    }
    __syncthreads();
    if (__syncthreads_or(long_run(s_kv, n, threadIdx.x, GS_BLOCK))) {
        block_sort_tile64(t, start, n, skey, pvals, s_kv, pair_emit, vals, keys64);
        return;
    }
    place_runs(t, start, n, s_kv, pvals, threadIdx.x, GS_BLOCK, pair_emit, vals, keys64);
    __syncthreads();
}

// Per-tile depth sort, a persistent grid over the dispatch records.  The
// first n_long records (kWaveSortMax<FEW> pairs or more) go to whole workgroups,
// records b, b + G, .. to workgroup b; then the waves take the rest, longest first,
// dealt out from the workgroup behind the last long tile's on: wave w of workgroup b
// records n_long + s for s = 4 ((b - n_long) mod G) + w and on in steps of 4G.
// Output: the tiles' pairs ordered by (depth bits, emission position), with
// the primitive ids, the sorted -> emission map and the optional 64-bit keys.
template <bool FEW>
__global__ void __launch_bounds__(GS_BLOCK) k_tile_depth_sort(const uint4* __restrict__ rec,
                                                              const uint32_t* __restrict__ n_long_ptr, uint32_t T,
                                                              PairRec* __restrict__ skey,
                                                              const uint32_t* __restrict__ pvals,
                                                              uint32_t* __restrict__ pair_emit,
                                                              uint32_t* __restrict__ vals,
                                                              uint64_t* __restrict__ keys64) {
    __shared__ unsigned long long s_kv[kLongCap];      // long tiles; a quarter per wave otherwise
    __shared__ uint32_t s_first[kSortWaves];
    const uint32_t G = gridDim.x;                             // <= T
    const uint32_t w = threadIdx.x / GS_WAVE;
    // the first record of the block loads beside the count
    uint4 rl = rec[blockIdx.x];
    const uint32_t n_long = *n_long_ptr;
    // the short tiles are dealt out, longest first, from the workgroups on that hold
    // no long tile (or the fewest): those with one get the shortest tiles, or none
    const uint32_t turn = n_long % G;
    const uint32_t s0 = (blockIdx.x >= turn ? blockIdx.x - turn : blockIdx.x + G - turn) * kSortWaves + w;
    uint4 rs = rec[min(n_long + s0, T - 1u)];
    for (uint32_t pos = blockIdx.x; pos < n_long; pos += G) {
        if (pos != blockIdx.x) rl = rec[pos];
        if (FEW && rl.z <= 2u * GS_BLOCK)
            sort_long_tile<2>(rl.x, rl.y, rl.z, skey, pvals, s_kv, s_first, pair_emit, vals, keys64);
        else if (FEW && rl.z <= 4u * GS_BLOCK)
            sort_long_tile<4>(rl.x, rl.y, rl.z, skey, pvals, s_kv, s_first, pair_emit, vals, keys64);
        else if (rl.z <= kLongCap)
            sort_long_tile<8>(rl.x, rl.y, rl.z, skey, pvals, s_kv, s_first, pair_emit, vals, keys64);
        else
            sort_huge_tile(rl.x, rl.y, rl.z, skey, pvals, s_kv, pair_emit, vals, keys64);
    }
    unsigned long long* sk = s_kv + w * (kLongCap / kSortWaves);
    for (uint32_t s = s0; s < T - n_long; s += kSortWaves * G) {
        if (s != s0) rs = rec[n_long + s];
        const uint32_t t = rs.x, start = rs.y, n = rs.z;
        if (n == 0u || n >= kWaveSortMax<FEW>) continue;     // (the order puts every longer tile first)
        if (n <= 64u)
            wave_sort_tile<1>(t, start, n, skey, pvals, sk, pair_emit, vals, keys64);
        else if (n <= 128u)
            wave_sort_tile<2>(t, start, n, skey, pvals, sk, pair_emit, vals, keys64);
        else if (FEW || n <= 256u)
            wave_sort_tile<4>(t, start, n, skey, pvals, sk, pair_emit, vals, keys64);
        else
            wave_sort_tile<8>(t, start, n, skey, pvals, sk, pair_emit, vals, keys64);
    }
}

struct BinsortLayout {
    size_t pkeys, emit_id;    // per emission position: tile and primitive of the pair
    size_t pdepth;            // per emission position: the primitive's depth bits
    size_t skey;              // per sorted position, a record: the 64-bit depth-sort key, the primitive
    size_t order;             // the dispatch order when the caller keeps none
    size_t rec;               // per dispatch position: tile, range start, pair count
    size_t tcount, cursor;    // per tile: pair total, placement cursor
    size_t bsum, offs, bstart, counters;
    size_t bytes;
};

uint32_t tile_count(int32_t width, int32_t height) {
    const int64_t TX = (width + GS_TILE - 1) / GS_TILE, TY = (height + GS_TILE - 1) / GS_TILE;
    return (uint32_t)(TX * TY);
}

BinsortLayout binsort_layout(int32_t n, uint32_t capacity, int32_t width, int32_t height) {
    BinsortLayout L;
    size_t o = 0;
    const size_t nn = (size_t)(n > 0 ? n : 1), cc = (size_t)(capacity > 0 ? capacity : 1);
    const size_t tt = (size_t)(width > 0 && height > 0 ? tile_count(width, height) : 1u);
    L.pkeys = o; o += align256(4 * cc);
    L.emit_id = o; o += align256(4 * cc);
    L.pdepth = o; o += align256(4 * cc);
    L.skey = o; o += align256(sizeof(PairRec) * cc);
    L.order = o; o += align256(4 * tt);
    L.rec = o; o += align256(16 * tt);
    L.tcount = o; o += align256(4 * tt);
    L.cursor = o; o += align256(4 * tt);
    L.bsum = o; o += align256(4 * ((size_t)div_up(nn, GS_TILE_ITEMS) + 1));
    L.offs = o; o += align256(4 * (nn + 1));
    L.bstart = o; o += align256(4 * ((size_t)div_up(cc, GS_TILE_ITEMS) + 1));
    L.counters = o; o += 256;
    L.bytes = o;
    return L;
}

template <typename T>
T* at(void* ws, size_t off) { return reinterpret_cast<T*>(static_cast<char*>(ws) + off); }

}  // namespace

size_t binsort_ws_bytes(int32_t n, uint32_t capacity, int32_t width, int32_t height) {
    return binsort_layout(n, capacity, width, height).bytes;
}

hipError_t launch_binsort(const gs_proj& proj, int32_t n, const uint32_t* vis_idx, const uint32_t* vis_count,
                          int32_t width, int32_t height, uint32_t capacity, uint32_t* vals, uint32_t* ranges,
                          uint32_t* tile_order, uint32_t* pair_offset, uint32_t* pair_emit, uint64_t* keys,
                          uint32_t* num_pairs, gs_device_status* status, void* ws, hipStream_t st) {
    const BinsortLayout L = binsort_layout(n, capacity, width, height);
    const int32_t TX = (width + GS_TILE - 1) / GS_TILE;
    const uint32_t T = tile_count(width, height);
    uint32_t* bsum = at<uint32_t>(ws, L.bsum);
    uint32_t* ctr = at<uint32_t>(ws, L.counters);   // [1] sort count, [2] long tiles
    uint32_t* tcount = at<uint32_t>(ws, L.tcount);
    uint32_t* cursor = at<uint32_t>(ws, L.cursor);
    uint32_t* order = tile_order ? tile_order : at<uint32_t>(ws, L.order);
    const uint32_t cus = compute_units() ? compute_units() : 256u;
    const bool few = T <= 2u * cus;
    // ranges, cursors and the dispatch order from the per-tile totals
    auto finish = [&]() {
        hipLaunchKernelGGL(k_tile_finish, dim3(div_up(T, kFinishSeg)), dim3(GS_BLOCK), 0, st, tcount, T, ranges,
                           cursor, order, at<uint4>(ws, L.rec), few ? kLongKey<true> : kLongKey<false>, ctr + 2);
        return hipGetLastError();
    };
    // no pairs: empty ranges, and the order (then the tile ids)
    auto no_pairs = [&]() {
        if (T == 0) return hipGetLastError();
        hipError_t e = launch_fill_u32(tcount, 0u, T, st);
        if (e != hipSuccess) return e;
        return finish();
    };
    if (n == 0) {
        hipError_t e = launch_fill_u32(num_pairs, 0u, 1, st);
        if (e != hipSuccess) return e;
        return no_pairs();
    }
    // 1. emission offsets in visible-set order
    const uint32_t* vorder = vis_idx;
    const uint32_t nb = div_up(n, GS_TILE_ITEMS);
    hipLaunchKernelGGL(k_tile_sums, dim3(nb), dim3(GS_BLOCK), 0, st, vorder, vis_count, proj.tiles, bsum, tcount, T);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    uint32_t* offs_r = at<uint32_t>(ws, L.offs);
    const uint32_t nbs = div_up(capacity, GS_TILE_ITEMS) + 1u;
    hipLaunchKernelGGL(k_offsets, dim3(nb), dim3(GS_BLOCK), 0, st, vorder, vis_count, proj.tiles, bsum, capacity, pair_offset, offs_r, ctr + 1, num_pairs, status, at<uint32_t>(ws, L.bstart), nbs);
    if (capacity == 0 || T == 0) return no_pairs();
    // 2. emission: one (tile, primitive) pair per touched tile, and the per-tile totals
    const uint32_t nbp = div_up(capacity, GS_TILE_ITEMS);
    hipLaunchKernelGGL(k_emit_pairs, dim3(nbp), dim3(GS_BLOCK), 0, st, vorder, vis_count, offs_r,
                       at<uint32_t>(ws, L.bstart), reinterpret_cast<const ushort4*>(proj.rect), proj.depth, ctr + 1,
                       TX, T, at<uint32_t>(ws, L.pkeys), at<uint32_t>(ws, L.emit_id), at<uint32_t>(ws, L.pdepth),
                       tcount);
    // 3. tile ranges and the dispatch order
    e = finish();
    if (e != hipSuccess) return e;
    // 4. every pair's depth-sort key placed in its tile's range
    PairRec* skey = at<PairRec>(ws, L.skey);
    const uint32_t* pvals = at<uint32_t>(ws, L.emit_id);
    hipLaunchKernelGGL(k_tile_scatter, dim3(nbp), dim3(GS_BLOCK), 0, st, at<uint32_t>(ws, L.pkeys),
                       pvals, at<uint32_t>(ws, L.pdepth), ctr + 1, T, cursor, skey);
    // 5. per tile, longest first: depth order, primitive ids (+ optional 64-bit keys)
    const dim3 grid(std::min<uint32_t>(T, cus * kDepthSortBlocksPerCU));
    if (few)
        hipLaunchKernelGGL(k_tile_depth_sort<true>, grid, dim3(GS_BLOCK), 0, st, at<uint4>(ws, L.rec), ctr + 2, T, skey,
                           pvals, pair_emit, vals, keys);
    else
        hipLaunchKernelGGL(k_tile_depth_sort<false>, grid, dim3(GS_BLOCK), 0, st, at<uint4>(ws, L.rec), ctr + 2, T, skey,
                           pvals, pair_emit, vals, keys);
    return hipGetLastError();
}

}  // namespace gsmi
