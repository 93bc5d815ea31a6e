// Binning of footprints into 16x16 tiles and the stable (tile, depth) sort.
//
// Entries are emitted in particle order, which is the tie order of the (tile, depth) sort, and
// a particle has at most one entry in a tile: inside a tile the stable depth order is the order
// of the 64-bit keys (depth bits, packed particle index), whatever order the entries arrive in.
// So the entries are placed straight into their tile's segment, in any order, and every segment
// is then sorted on that key; no global radix passes carry the entries through memory.
//
// Steps (all on the caller's stream, no host synchronisation):
//   1. count      a workgroup takes a chunk of a view's particles and counts its entries per
//                 tile in LDS; the counts are one row of the view's (chunk, tile) matrix
//   2. columns    per tile, the exclusive prefix over the chunks and the total; 64-tile sums
//   3. top        scans of the 64-tile sums and of the chunks' entry totals, count, status
//   4. place      the chunk again: emit offsets, and every entry (key) to its tile's segment at
//                 the chunk's position in it plus an LDS counter; tile ranges, and the segments
//                 of more than kSmallMax entries listed by size
//   5. partition  segments longer than kBigMax: distributed over buckets of the depth range
//                 until every piece fits the sort of step 6
//   6. sort       segments and pieces in LDS: one wave, four waves or sixteen waves each
#include "common.h"
#include <algorithm>

#include "kernels.h"

namespace isogs {

constexpr int kBinThreads = 1024;
constexpr int kBinWaves = kBinThreads / kWave;
constexpr uint32_t kColTiles = 64;                      // tiles per column-scan workgroup
constexpr uint32_t kMaxChunks = 512;                    // rows of a view's matrix at most
// tiles a workgroup counts at once (one LDS word each): views of up to 1080p, and larger ones
// (4K has 32400) with one workgroup per CU; a view with more tiles is taken in bands. Two
// workgroups of 18432 tiles would fit a CU as well: 2560 x 1440 views of 1M particles take 114 us
// with either, two 166, ten 712 and 715, and only four (358 and 334, by the chunks of that build)
// differ.
constexpr uint32_t kBandSmall = 9216, kBandLarge = 36864;
constexpr uint32_t kSmallMax = 256;                     // sorted by one wave
constexpr uint32_t kMidMax = 1024;                      // by four
constexpr uint32_t kBigMax = 4096;                      // by sixteen
constexpr uint32_t kCountLimit = (1u << 30) - 1u;       // entries per batch must stay below
constexpr uint64_t kGroupMaxParticles = 131072;         // calls of up to so many: eight lanes per particle

// A view's place in the binning arrays.
struct BinView {
    uint32_t p_off, n;                  // packed particles
    uint32_t tile_base, tiles;          // global tiles
    int32_t width, height, tiles_x, tiles_y;
    uint32_t per, chunks, chunk0;       // particles per chunk, chunks, index of the first
    uint32_t block0;                    // its first 64-tile block
    uint64_t m_off;                     // its matrix: [chunks][tiles + 1] counts
};

struct BinPack {
    int32_t nv;
    uint32_t view0;                        // index of the launch's first view
    uint32_t chunk_begin[kMaxViews + 1];   // chunks of earlier views in this launch
    uint32_t block_begin[kMaxViews + 1];   // column-scan blocks of earlier views
    uint32_t tile0, tiles;                 // global tiles of the launch
    uint32_t bands;                        // of its view with the most tiles
    uint32_t miss_pitch;
    uint32_t* miss;                        // [chunks][miss_pitch] entries without a tile (views of several bands)
    BinView v[kMaxViews];
};

// A piece of a segment (sorted by step 6): its entries, tile and the buffer that holds it
// (0: the keys, 1: depth bits in the workspace and indices in pidx).
struct SortItem {
    uint32_t start, n, tile, buf;
};

// Counters, one per 128-byte line.
constexpr uint32_t kLine = 32;
enum : uint32_t { kNumMid = 0, kNumBig = kLine, kNumLarge = 2 * kLine, kWork = 3 * kLine, kNumMidItems = 4 * kLine,
                  kNumBigItems = 5 * kLine, kCounterWords = 6 * kLine };

// Device arrays of one call.
struct BinArrays {
    uint64_t* key;          // [capacity] (depth bits << 32) | packed particle index, by tile
    uint32_t* z_alt;        // [capacity] the other buffer's depth bits (its indices are in pidx)
    uint2* box;             // [N] tile boxes of step 1 for step 4, or NULL
    uint32_t* m;            // the (chunk, tile) matrices
    uint32_t* tile_pre;     // [T] entries of the 64-tile block's earlier tiles
    uint32_t* tile_tot;     // [T]
    uint32_t* missing;      // [views] entries without a tile
    uint32_t* missing_at;   // [views] and their first position
    uint32_t* block_sum;    // [64-tile blocks], scanned by step 3
    uint64_t* chunk_sum;    // [chunks], scanned by step 3
    uint32_t* counters;
    uint32_t *mid, *big;    // tiles listed by segment length
    SortItem *large, *mid_item, *big_item;
    uint2* stack;           // pending ranges of step 5: slots start / 4096 .. of each segment
    uint32_t list_max, large_max, item_max;
    uint32_t blocks, chunks, views;
};

// Inclusive scan over the 64 lanes of a wave: DPP shifts inside the four 16-lane rows, then the
// totals of the earlier rows as scalars (shuffles through LDS cost a round trip per step).
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15), r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31),
                   r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
    const uint32_t row = lane_id() >> 4;
    return x + (row == 0 ? 0u : row == 1 ? r0 : row == 2 ? r0 + r1 : r0 + r1 + r2);
}

__device__ __forceinline__ uint64_t wave_inclusive_scan(uint64_t x) {
    const int lane = (int)lane_id();
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint64_t y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    return x;
}

// Largest value of the wave, in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true));
    return max(max((uint32_t)__builtin_amdgcn_readlane((int)x, 15), (uint32_t)__builtin_amdgcn_readlane((int)x, 31)),
               max((uint32_t)__builtin_amdgcn_readlane((int)x, 47), (uint32_t)__builtin_amdgcn_readlane((int)x, 63)));
}

// Exclusive scan over a block of NW waves; s_tmp holds NW words. Returns the block total
// in `total`. Contains __syncthreads.
template <int NW, typename T>
__device__ __forceinline__ T block_exclusive_scan(T x, T* s_tmp, T& total) {
    const uint32_t w = threadIdx.x >> 6;
    const T inc = wave_inclusive_scan(x);
    if (lane_id() == kWave - 1) s_tmp[w] = inc;
    __syncthreads();
    T before = 0;
    total = 0;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        before += ((uint32_t)j < w) ? s_tmp[j] : (T)0;
        total += s_tmp[j];
    }
    __syncthreads();
    return before + inc - x;
}

// Orders the LDS accesses of a wave before and after (the hardware completes a wave's LDS
// operations in order; this holds the compiler to it).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- Tile boxes -----------------------------------------------------------------------------

// The candidate tiles of a particle, row-major cells of a w x h box.
struct TileBox {
    float u, v, r2, w_lim, h_lim;
    int tx0, ty0, w, h;
    __device__ bool member(int cx, int cy) const { return tile_member(u, v, r2, tx0 + cx, ty0 + cy, w_lim, h_lim); }
    // the tiles of the view from its first cell to its last (an empty box: tile 0)
    __device__ uint2 span(const BinView& vd) const {
        const uint32_t first = (uint32_t)(ty0 * vd.tiles_x + tx0);
        return w ? make_uint2(first, first + (uint32_t)((h - 1) * vd.tiles_x + w - 1)) : make_uint2(0u, 0u);
    }
};

// What a particle's box is made of.
struct BoxLoad {
    float u, v, r;
};
__device__ __forceinline__ BoxLoad load_footprint(const float4* __restrict__ record, uint32_t i) {
    const float2 uv = *reinterpret_cast<const float2*>(record + 2 * (size_t)i);
    return {uv.x, uv.y, record[2 * (size_t)i + 1].w};
}

__device__ __forceinline__ TileBox make_box(const BinView& vd, const BoxLoad& l) {
    const float r = l.r;
    TileBox b;
    b.u = l.u;
    b.v = l.v;
    b.r2 = r * r;
    b.w_lim = (float)vd.width - 0.5f;
    b.h_lim = (float)vd.height - 0.5f;
    int tx1, ty1;
    tile_box(l.u, l.v, r, vd.tiles_x, vd.tiles_y, b.tx0, tx1, b.ty0, ty1);
    b.w = max(0, tx1 - b.tx0 + 1);
    b.h = max(0, ty1 - b.ty0 + 1);
    if (b.w == 0 || b.h == 0) b.w = b.h = 0;
    return b;
}

// A box of at most 4 x 4 cells with its members as a bit mask (bit 4 y + x), in 8 bytes: step 4
// then reads 8 bytes of a particle instead of its 32-byte record, and visits members only. The
// squared offsets of four columns and four rows are formed once, so that a wave does not go
// through as many turns as its largest box has cells. Any other box (larger, a tile coordinate
// of 4096 or more, a tile count other than its members') is marked and walked again.
constexpr uint32_t kBoxWalk = 0x80000000u;
__device__ __forceinline__ uint32_t box_mask4(const TileBox& b) {
    float dxx[4], dyy[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // (tile_member's arithmetic)
        const float x0 = (float)((b.tx0 + q) * kTile), y0 = (float)((b.ty0 + q) * kTile);
        const float dx = fmaxf(fmaxf(x0 + 0.5f - b.u, b.u - fminf(x0 + 15.5f, b.w_lim)), 0.0f);
        const float dy = fmaxf(fmaxf(y0 + 0.5f - b.v, b.v - fminf(y0 + 15.5f, b.h_lim)), 0.0f);
        dxx[q] = dx * dx;
        dyy[q] = dy * dy;
    }
    uint32_t mask = 0;
#pragma unroll
    for (int c = 0; c < 16; ++c) mask |= (dxx[c & 3] + dyy[c >> 2] <= b.r2 ? 1u : 0u) << c;
    // cells of the box only
    return mask & ((1u << min(b.w, 4)) - 1u) * 0x1111u & ((1u << 4 * min(b.h, 4)) - 1u);
}

// Calls put(tile of the view) for the members of a mask whose cell 0 is tile `first`.
template <typename Fn>
__device__ __forceinline__ void put_mask4(uint32_t mask, uint32_t first, uint32_t tiles_x, Fn put) {
    while (mask) {
        const uint32_t c = (uint32_t)__ffs((int)mask) - 1u;
        mask &= mask - 1u;
        put(first + (c >> 2) * tiles_x + (c & 3u));
    }
}

// Calls put(tile of the view) for the first `want` members of a box of any size, by the group
// of G lanes (lane j of it) that holds the particle. Returns their number in every lane.
template <int G, typename Fn>
__device__ __forceinline__ uint32_t walk_box(const BinView& vd, const TileBox& b, uint32_t want, uint32_t j, Fn put) {
    uint32_t n = 0;
    if (G > 1) {
        // count together, then place together; a count below the members (the tile count came
        // from elsewhere) is placed by the first lane alone, in order
        const uint32_t cells = (uint32_t)(b.w * b.h);
        int cx = (int)j, cy = 0;
        for (uint32_t c = j; c < cells; c += G, cx += G) {
            while (cx >= b.w) {
                cx -= b.w;
                ++cy;
            }
            n += b.member(cx, cy) ? 1u : 0u;
        }
#pragma unroll
        for (int o = 1; o < G; o <<= 1) n += __shfl_xor(n, o, kWave);
        if (n <= want) {
            cx = (int)j;
            cy = 0;
            for (uint32_t c = j; c < cells; c += G, cx += G) {
                while (cx >= b.w) {
                    cx -= b.w;
                    ++cy;
                }
                if (b.member(cx, cy)) put((uint32_t)((b.ty0 + cy) * vd.tiles_x + b.tx0 + cx));
            }
            return n;
        }
        if (j != 0) return want;
        n = 0;
    }
    for (int y = 0; y < b.h && n < want; ++y)
        for (int x = 0; x < b.w && n < want; ++x)
            if (b.member(x, y)) {
                ++n;
                put((uint32_t)((b.ty0 + y) * vd.tiles_x + b.tx0 + x));
            }
    return n;
}

// Members of a box up to `want`, counted by one lane.
__device__ __forceinline__ uint32_t count_members(const TileBox& b, uint32_t want) {
    uint32_t n = 0;
    for (int y = 0; y < b.h && n < want; ++y)
        for (int x = 0; x < b.w && n < want; ++x) n += b.member(x, y) ? 1u : 0u;
    return n;
}

// Chunk and band of workgroup b of work_blocks: the bands of a chunk, which read the same
// particles, follow each other on one XCD (b mod 8). Eight chunks at a time, some past the last;
// of fewer than kXcdChunks that would leave XCDs idle. 6M particles in 5120 x 2880: 519 -> 497 us,
// in 7680 x 4320 779 -> 734; with 28 chunks on eight XCDs 12288 x 6912 took 1569 us against 1327.
constexpr uint32_t kXcdChunks = 32;
struct ChunkBand {
    uint32_t chunk, band;
};
__host__ __device__ constexpr uint32_t work_blocks(uint32_t chunks, uint32_t bands) {
    return bands == 1 ? chunks : (chunks >= kXcdChunks ? (chunks + 7u) / 8u * 8u : chunks) * bands;
}
template <bool BANDED>
__device__ __forceinline__ ChunkBand chunk_band(uint32_t b, uint32_t chunks, uint32_t bands) {
    if (!BANDED || bands == 1) return {b, 0u};
    if (chunks < kXcdChunks) return {b % chunks, b / chunks};
    const uint32_t group = b / (8u * bands), in = b - group * 8u * bands;
    return {8u * group + (in & 7u), in >> 3};
}

__device__ __forceinline__ int view_of_chunk(const BinPack& pk, uint32_t b) {
    int v = 0;
    for (int i = 1; i < pk.nv; ++i) v = (b >= pk.chunk_begin[i]) ? i : v;
    return __builtin_amdgcn_readfirstlane(v);
}

// A wave's particles whose boxes reach into the workgroup's band, gathered until there is one per
// lane: a view of many bands has few of any 64 particles in one of them, and a wave walks as long
// for one particle as for 64. From kQueueDirect lanes on they are walked where they are, which
// saves loading them again. Bin sort of one view, walked by every band and ungathered before,
// and now: 1M particles, 7680 x 4320, 428 -> 273 us, 12288 x 6912 1.40 -> 0.47 ms, 16384 x 16384
// 11.4 -> 1.7 ms; 300k in 32768 x 32768 130 -> 5.3 ms. From 8 lanes on 12288 x 6912 takes 664 us,
// from 16 521; never, 477, but 6M particles in 7680 x 4320 724 us against 685.
constexpr int kQueueDirect = 24;
struct BoxQueue {
    uint32_t* at;        // this wave's 2 kWave words of LDS
    uint32_t held = 0;   // uniform over the wave
    // Adds `value` of the lanes with `in`; calls fn(value) for the G lanes of each particle taken.
    // Where enough of the wave is in, now() walks those at once.
    template <int G, typename Fn, typename Now>
    __device__ __forceinline__ void add(bool in, uint32_t value, Fn fn, Now now) {
        const uint64_t m = ballot64(in);
        if (G == 1 && __popcll(m) >= kQueueDirect) {   // uniform
            if (in) now();
            return;
        }
        if (in) at[held + rank_below(m)] = value;
        held += (uint32_t)__popcll(m);
        if (held < (uint32_t)kWave) return;   // uniform
        held -= kWave;
        take<G>(held, kWave, fn);
    }
    template <int G, typename Fn>
    __device__ __forceinline__ void end(Fn fn) {
        take<G>(0, held, fn);
    }

private:
    template <int G, typename Fn>
    __device__ __forceinline__ void take(uint32_t from, uint32_t n, Fn fn) {
        wave_lds_order();
        for (uint32_t q = lane_id() / G; q < n; q += kWave / G) fn(at[from + q]);
        wave_lds_order();
    }
};

// Step 1. A particle has no more entries than its tile count says; missing ones (the count may
// come from elsewhere) belong to no tile and go behind all others. G lanes share a particle
// (small scenes: few particles, large boxes). Bound by the records' bytes and the walk over the box.
// BANDED: a view of the call has several bands. Each of them reads every particle and walks those
// that reach into it, and the band of a box's first tile counts its missing entries and keeps its
// packed form.
template <uint32_t BT, int G, bool BANDED>
__global__ void __launch_bounds__(kBinThreads) bin_count_kernel(const BinPack pk, const float4* __restrict__ record,
                                                                const uint32_t* __restrict__ tile_count,
                                                                const BinArrays A) {
    __shared__ uint32_t s_h[BT];
    __shared__ unsigned long long s_sum;
    __shared__ uint32_t s_miss;
    constexpr uint32_t kStep = BANDED ? kBinThreads : kBinThreads / G;   // particles per turn
    const uint32_t t = threadIdx.x, j = t % G;
    const ChunkBand cb = chunk_band<BANDED>(blockIdx.x, pk.chunk_begin[pk.nv], pk.bands);
    if (BANDED && cb.chunk >= pk.chunk_begin[pk.nv]) return;
    const int vi = view_of_chunk(pk, cb.chunk);
    const BinView& vd = pk.v[vi];
    const uint32_t row = cb.chunk - pk.chunk_begin[vi], t0 = cb.band * BT;
    if (t0 >= vd.tiles && cb.band) return;   // (uniform) fewer bands than the launch's largest view
    const uint32_t nt = min(BT, vd.tiles - t0);
    for (uint32_t q = t; q < nt; q += kBinThreads) s_h[q] = 0u;
    if (t == 0) {
        s_sum = 0;
        s_miss = 0;
    }
    __syncthreads();
    const uint32_t c0 = row * vd.per, c1 = min(vd.n, c0 + vd.per);
    unsigned long long sum = 0;
    uint32_t miss = 0;
    // one particle, by its G lanes
    auto walk = [&](uint32_t g, uint32_t want, const TileBox& b) {
        auto put = [&](uint32_t tile) {
            if (tile - t0 < nt) atomicAdd(&s_h[tile - t0], 1u);
        };
        const uint2 span = BANDED ? b.span(vd) : make_uint2(0u, 0u);
        uint2 packed = make_uint2(span.x, kBoxWalk | span.y);
        uint32_t n;
        const uint32_t mask = b.w <= 4 && b.h <= 4 ? box_mask4(b) : 0u;
        if ((uint32_t)__popc(mask) == want && (b.tx0 | b.ty0) < 4096) {
            n = want;
            packed = make_uint2(mask, (uint32_t)b.tx0 | (uint32_t)b.ty0 << 12);
            if (j == 0) put_mask4(mask, (uint32_t)(b.ty0 * vd.tiles_x + b.tx0), (uint32_t)vd.tiles_x, put);
        } else {
            n = walk_box<G>(vd, b, want, j, put);
        }
        if (j == 0 && (!BANDED || span.x - t0 < nt)) {
            miss += want - n;
            if (A.box) A.box[g] = packed;
        }
    };
    // the next particle is loaded while this one is walked (past the end: the last one again)
    const uint32_t mine = BANDED ? t : t / G;
    const uint32_t last = vd.p_off + max(c1, 1u) - 1u, first = vd.p_off + c0 + mine;
    BoxLoad next_box{0.0f, 0.0f, 0.0f};
    uint32_t next_want = 0;
    if (c0 < c1) {
        next_box = load_footprint(record, min(first, last));
        next_want = tile_count[min(first, last)];
    }
    auto next = [&](uint32_t i, BoxLoad& load, uint32_t& want) {
        const uint32_t g = vd.p_off + i;
        load = next_box;
        want = i < c1 ? next_want : 0u;
        next_box = load_footprint(record, min(g + kStep, last));
        next_want = tile_count[min(g + kStep, last)];
    };
    BoxLoad load;
    uint32_t want;
    if constexpr (BANDED) {
        __shared__ uint32_t s_queue[kBinWaves][2 * kWave];
        BoxQueue queue{s_queue[t >> 6]};
        auto gathered = [&](uint32_t g) { walk(g, tile_count[g], make_box(vd, load_footprint(record, g))); };
        for (uint32_t q = c0; q < c1; q += kStep) {
            const uint32_t g = vd.p_off + q + t;
            next(q + t, load, want);
            const uint2 span = make_box(vd, load).span(vd);
            sum += want;
            queue.add<G>(want && span.x < t0 + nt && span.y >= t0, g, gathered,
                         [&] { walk(g, want, make_box(vd, load)); });
        }
        queue.end<G>(gathered);
    } else {
        for (uint32_t q = c0; q < c1; q += kStep) {
            next(q + mine, load, want);
            if (!want) continue;   // whole groups
            walk(vd.p_off + q + mine, want, make_box(vd, load));
            if (j == 0) sum += want;
        }
    }
    if (sum && cb.band == 0) atomicAdd(&s_sum, sum);
    if (miss) atomicAdd(&s_miss, miss);
    __syncthreads();
    uint32_t* m = A.m + vd.m_off + (size_t)row * (vd.tiles + 1);
    for (uint32_t q = t; q < nt; q += kBinThreads) m[t0 + q] = s_h[q];
    if (t == 0) {
        if (cb.band == 0) A.chunk_sum[vd.chunk0 + row] = s_sum;
        if (BANDED)
            pk.miss[(size_t)(vd.chunk0 + row) * pk.miss_pitch + cb.band] = s_miss;
        else
            m[vd.tiles] = s_miss;
    }
}

// Step 2: 64 columns (tiles; the last column of a view holds the entries without a tile) per
// workgroup, a wave per run of up to kMaxChunks / 16 rows held in registers.
template <bool BANDED>
__global__ void __launch_bounds__(kBinThreads) bin_columns_kernel(const BinPack pk, const BinArrays A) {
    __shared__ uint32_t s_part[kBinWaves][kColTiles];
    constexpr uint32_t kRows = kMaxChunks / kBinWaves;
    int v = 0;
    for (int i = 1; i < pk.nv; ++i) v = (blockIdx.x >= pk.block_begin[i]) ? i : v;
    v = __builtin_amdgcn_readfirstlane(v);
    const BinView& vd = pk.v[v];
    const uint32_t w = threadIdx.x >> 6, l = lane_id();
    const uint32_t block = blockIdx.x - pk.block_begin[v], col = block * kColTiles + l;
    const uint32_t rows = (vd.chunks + kBinWaves - 1) / kBinWaves, r0 = w * rows;
    uint32_t* m = A.m + vd.m_off + col;
    const size_t pitch = vd.tiles + 1;
    const bool on = col <= vd.tiles;
    uint32_t x[kRows], sum = 0;
#pragma unroll
    for (uint32_t r = 0; r < kRows; ++r) x[r] = on && r < rows && r0 + r < vd.chunks ? m[(r0 + r) * pitch] : 0u;
    if (BANDED && col == vd.tiles) {   // the entries without a tile are kept by band
        const uint32_t bands = (vd.tiles + kBandLarge - 1) / kBandLarge;
#pragma unroll
        for (uint32_t r = 0; r < kRows; ++r) {
            x[r] = 0u;
            if (r >= rows || r0 + r >= vd.chunks) continue;
            for (uint32_t b = 0; b < bands; ++b) x[r] += pk.miss[(size_t)(vd.chunk0 + r0 + r) * pk.miss_pitch + b];
        }
    }
#pragma unroll
    for (uint32_t r = 0; r < kRows; ++r) sum += x[r];
    s_part[w][l] = sum;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (uint32_t q = 0; q < (uint32_t)kBinWaves; ++q) {
        const uint32_t y = s_part[q][l];
        run += q < w ? y : 0u;
        total += y;
    }
#pragma unroll
    for (uint32_t r = 0; r < kRows; ++r) {
        if (on && r < rows && r0 + r < vd.chunks) m[(r0 + r) * pitch] = run;
        run += x[r];
    }
    if (w != 0) return;
    const uint32_t mine = col < vd.tiles ? total : 0u;
    const uint32_t incl = wave_inclusive_scan(mine);
    if (col < vd.tiles) {
        A.tile_pre[vd.tile_base + col] = incl - mine;
        A.tile_tot[vd.tile_base + col] = total;
    }
    if (col == vd.tiles) A.missing[pk.view0 + v] = total;
    if (l == kWave - 1) A.block_sum[vd.block0 + block] = incl;
}

// Exclusive scan of v[0, n) (values T) by one workgroup, in place or into `out`, starting
// from `base`; returns base plus the total. Contains __syncthreads.
template <typename T, typename O>
__device__ __forceinline__ uint64_t scan_array(const T* v, O* out, uint32_t n, uint64_t base, uint64_t* s_tmp) {
    const uint32_t per = (n + kBinThreads - 1) / kBinThreads;
    const uint32_t i0 = min(n, threadIdx.x * per), i1 = min(n, i0 + per);
    uint64_t sum = 0;
    for (uint32_t i = i0; i < i1; ++i) sum += v[i];
    uint64_t total;
    uint64_t run = base + block_exclusive_scan<kBinWaves, uint64_t>(sum, s_tmp, total);
    for (uint32_t i = i0; i < i1; ++i) {
        const T x = v[i];
        out[i] = (O)run;
        run += x;
    }
    return base + total;
}

// Step 3: one workgroup.
__global__ void __launch_bounds__(kBinThreads) bin_top_kernel(const BinArrays A, uint64_t capacity,
                                                              uint32_t* __restrict__ count,
                                                              int32_t* __restrict__ status) {
    __shared__ uint64_t s_tmp[kBinWaves];
    if (threadIdx.x < kCounterWords) A.counters[threadIdx.x] = 0u;
    const uint64_t in_tiles = scan_array(A.block_sum, A.block_sum, A.blocks, 0, s_tmp);
    scan_array(A.missing, A.missing_at, A.views, in_tiles, s_tmp);
    const uint64_t total = scan_array(A.chunk_sum, A.chunk_sum, A.chunks, 0, s_tmp);
    if (threadIdx.x == 0) {
        const bool fits = total <= capacity && total < (uint64_t)kCountLimit;
        *count = (uint32_t)(total > 0xFFFFFFFFull ? 0xFFFFFFFFull : total);
        *status = fits ? kStatusOk : kStatusCapacity;
    }
}

__device__ __forceinline__ uint32_t tile_start(const BinArrays& A, const BinView& vd, uint32_t tile) {
    return A.block_sum[vd.block0 + tile / kColTiles] + A.tile_pre[vd.tile_base + tile];
}

// Tile ranges of 1024 tiles, and the lists of those with more than kSmallMax entries (one
// device-wide add per workgroup and list). Contains __syncthreads.
__device__ __forceinline__ void bin_ranges(const BinPack& pk, const BinArrays& A, uint32_t block, bool ok,
                                           uint32_t* __restrict__ ranges) {
    __shared__ uint32_t s_n[3], s_at[3];
    const uint32_t t = threadIdx.x, i = block * kBinThreads + t;
    if (t < 3) s_n[t] = 0;
    __syncthreads();
    uint32_t start = 0, n = 0;
    if (i < pk.tiles && ok) {
        int v = 0;
        for (int q = 1; q < pk.nv; ++q) v = pk.tile0 + i >= pk.v[q].tile_base ? q : v;
        const BinView& vd = pk.v[v];
        n = A.tile_tot[pk.tile0 + i];
        start = n ? tile_start(A, vd, pk.tile0 + i - vd.tile_base) : 0u;
    }
    if (i < pk.tiles) {
        ranges[2 * (size_t)(pk.tile0 + i)] = start;
        ranges[2 * (size_t)(pk.tile0 + i) + 1] = start + n;
    }
    const uint32_t c = n <= kSmallMax ? 3u : n <= kMidMax ? 0u : n <= kBigMax ? 1u : 2u;
    uint32_t at = 0;
    if (c < 3u) at = atomicAdd(&s_n[c], 1u);
    __syncthreads();
    if (t < 3 && s_n[t]) s_at[t] = atomicAdd(&A.counters[t * kLine], s_n[t]);
    __syncthreads();
    if (c >= 3u) return;
    at += s_at[c];
    if (at >= (c == 2u ? A.large_max : A.list_max)) return;   // (the bound on tiles with so many entries)
    if (c == 0u) A.mid[at] = pk.tile0 + i;
    if (c == 1u) A.big[at] = pk.tile0 + i;
    if (c == 2u) A.large[at] = SortItem{start, n, pk.tile0 + i, 0u};
}

// Step 4. A workgroup takes a chunk and a band; those past them write tile ranges. The key writes
// are scattered: a chunk has a few entries for each of thousands of tiles, so they are bound by
// the caches' handling of partial lines rather than by bytes.
template <uint32_t BT, int G, bool BANDED>
__global__ void __launch_bounds__(kBinThreads) __attribute__((amdgpu_waves_per_eu(BT == kBandSmall ? 8 : 4))) bin_place_kernel(const BinPack pk, const float4* __restrict__ record,
                                                                const float* __restrict__ depth,
                                                                const uint32_t* __restrict__ tile_count,
                                                                const BinArrays A, const int32_t* __restrict__ status,
                                                                const uint32_t* __restrict__ count_p,
                                                                uint32_t* __restrict__ ranges,
                                                                uint32_t* __restrict__ offsets,
                                                                uint32_t* __restrict__ pidx) {
    __shared__ uint32_t s_c[BT];
    __shared__ uint32_t s_tmp[kBinWaves];
    const uint32_t t = threadIdx.x, j = t % G;
    const bool ok = *status == kStatusOk;
    const uint32_t n_chunks = pk.chunk_begin[pk.nv], n_work = BANDED ? work_blocks(n_chunks, pk.bands) : n_chunks;
    if (blockIdx.x >= n_work) {
        bin_ranges(pk, A, blockIdx.x - n_work, ok, ranges);
        return;
    }
    const ChunkBand cb = chunk_band<BANDED>(blockIdx.x, n_chunks, pk.bands);
    if (BANDED && cb.chunk >= n_chunks) return;
    const int vi = view_of_chunk(pk, cb.chunk);
    const BinView& vd = pk.v[vi];
    const uint32_t row = cb.chunk - pk.chunk_begin[vi], t0 = cb.band * BT;
    if (t0 >= vd.tiles && cb.band) return;
    const uint32_t nt = min(BT, vd.tiles - t0), count = *count_p;
    const uint32_t* m = A.m + vd.m_off + (size_t)row * (vd.tiles + 1);
    if (ok)
#pragma unroll(BT == kBandLarge ? 4 : 1)
        for (uint32_t q = t; q < nt; q += kBinThreads) s_c[q] = tile_start(A, vd, t0 + q) + m[t0 + q];
    const uint32_t c0 = row * vd.per, c1 = min(vd.n, c0 + vd.per);
    if (cb.band == 0) {
        // emit offsets, and the entries without a tile (emit order)
        const uint32_t n_missing = ok ? m[vd.tiles] : 0u;   // (of earlier chunks: a prefix)
        const bool any_missing = ok && A.missing[pk.view0 + vi] != 0u;
        uint32_t run = (uint32_t)A.chunk_sum[vd.chunk0 + row];
        uint32_t at = any_missing ? A.missing_at[pk.view0 + vi] + n_missing : 0u;
        for (uint32_t q = c0; q < c1; q += kBinThreads) {
            const uint32_t i = q + t, want = i < c1 ? tile_count[vd.p_off + i] : 0u;
            uint32_t total;
            const uint32_t o = run + block_exclusive_scan<kBinWaves, uint32_t>(want, s_tmp, total);
            if (i < c1) offsets[vd.p_off + i] = o;
            run += total;
            if (!any_missing) continue;   // uniform
            const uint32_t miss =
                want ? want - count_members(make_box(vd, load_footprint(record, vd.p_off + i)), want) : 0u;
            const uint32_t p = at + block_exclusive_scan<kBinWaves, uint32_t>(miss, s_tmp, total);
            for (uint32_t k = 0; k < miss && p + k < count; ++k) pidx[p + k] = vd.p_off + i;
            at += total;
        }
    }
    if (!ok || c0 >= c1) return;
    __syncthreads();
    // one particle, by its G lanes
    auto place = [&](uint32_t g, uint32_t want, uint32_t z, const uint2& b) {
        const uint64_t key = (uint64_t)z << 32 | g;
        auto put = [&](uint32_t tile) {
            if (tile - t0 >= nt) return;
            const uint32_t p = atomicAdd(&s_c[tile - t0], 1u);
            if (p < count) A.key[p] = key;
        };
        if (b.y & kBoxWalk)
            walk_box<G>(vd, make_box(vd, load_footprint(record, g)), want, j, put);
        else if (j == 0)
            put_mask4(b.x, (b.y >> 12) * (uint32_t)vd.tiles_x + (b.y & 0xFFFu), (uint32_t)vd.tiles_x, put);
    };
    constexpr uint32_t kStep = BANDED ? kBinThreads : kBinThreads / G;
    const uint32_t mine = BANDED ? t : t / G;
    const uint32_t last = vd.p_off + c1 - 1u, first = min(vd.p_off + c0 + mine, last);
    uint32_t next_want = tile_count[first], next_z = __float_as_uint(depth[first]);
    uint2 next_box = A.box ? A.box[first] : make_uint2(0u, kBoxWalk);
    if constexpr (BANDED) {
        __shared__ uint32_t s_queue[kBinWaves][2 * kWave];
        BoxQueue queue{s_queue[t >> 6]};
        auto gathered = [&](uint32_t g) {
            place(g, tile_count[g], __float_as_uint(depth[g]), A.box ? A.box[g] : make_uint2(0u, kBoxWalk));
        };
        for (uint32_t q = c0; q < c1; q += kStep) {
            const uint32_t g = vd.p_off + q + t, ahead = min(g + kStep, last);
            const uint32_t want = q + t < c1 ? next_want : 0u, z = next_z;
            const uint2 b = next_box;
            next_want = tile_count[ahead];
            next_z = __float_as_uint(depth[ahead]);
            if (A.box) next_box = A.box[ahead];
            uint2 span;
            if (!A.box) {
                span = make_box(vd, load_footprint(record, min(g, last))).span(vd);
            } else if (b.y & kBoxWalk) {
                span = make_uint2(b.x, b.y & ~kBoxWalk);
            } else {   // (four rows: no member lies beyond)
                span.x = (b.y >> 12) * (uint32_t)vd.tiles_x + (b.y & 0xFFFu);
                span.y = span.x + 3u * (uint32_t)vd.tiles_x + 3u;
            }
            queue.add<G>(want && span.x < t0 + nt && span.y >= t0, g, gathered,
                         [&] { place(g, want, z, b); });
        }
        queue.end<G>(gathered);
    } else {
        for (uint32_t q = c0; q < c1; q += kStep) {
            const uint32_t i = q + mine, g = vd.p_off + i, ahead = min(g + kStep, last);
            const uint32_t want = i < c1 ? next_want : 0u, z = next_z;
            const uint2 b = next_box;
            next_want = tile_count[ahead];
            next_z = __float_as_uint(depth[ahead]);
            if (A.box) next_box = A.box[ahead];
            if (want) place(g, want, z, b);   // whole groups
        }
    }
}

// ---- Sorting in LDS ---------------------------------------------------------------------------

// Where a piece is read from.
struct SortSource {
    const uint64_t* key;
    const uint32_t* z_alt;
    uint32_t buf;
    __device__ uint64_t at(uint32_t p, const uint32_t* pidx) const {
        return buf ? (uint64_t)z_alt[p] << 32 | pidx[p] : key[p];
    }
};

// Buckets: a monotone map of the depth bits (of the index where all depths are equal) from
// their range [lo, hi] to [0, nb): nb equal parts of the range.
struct BucketMap {
    uint32_t lo, nb;
    bool by_index;
    float scale;
    __device__ BucketMap(uint32_t lo_, uint32_t hi, bool by_index_, uint32_t nb_) : lo(lo_), nb(nb_), by_index(by_index_) {
        scale = (float)nb / ((float)(hi - lo) + 1.0f);
    }
    // position in units of buckets, and the bucket of a position
    __device__ float at(uint64_t k) const { return (float)((by_index ? (uint32_t)k : (uint32_t)(k >> 32)) - lo) * scale; }
    __device__ uint32_t bucket(float v) const { return min((uint32_t)v, nb - 1u); }
    __device__ uint32_t of(uint64_t k) const { return bucket(at(k)); }
};

// Sorted by THREADS threads (a wave, or the workgroup): up to THREADS * ITEMS entries. Entries
// are counted in 4 THREADS equal parts of the depth range; a part that holds c of them, the
// entries [base, base + c), is divided again into c buckets (the parts' counts are a
// piecewise linear distribution function, and every bucket takes an equal share of it: the
// depths of a tile lie in a few dense surfaces and clusters, and equal buckets of the range
// alone left dozens of entries in some). The buckets are counted and scanned, the entries stored
// by bucket, and an entry's rank inside its bucket is the number of smaller keys there, usually
// one or two reads. Six LDS round trips whatever the key width, where ranking three 8-bit digits by
// ballots took about 35 instructions per digit and entry. Where a bucket holds more than
// kBucketMax (many equal depths) the keys go through a bitonic network instead.
constexpr uint32_t kBucketMax = 64;

template <int THREADS, int ITEMS>
struct __align__(16) SortShared {
    union {
        uint64_t key[THREADS * ITEMS];
        uint32_t part[THREADS * 4 + 4];     // before the entries are stored
        uint32_t sorted[THREADS * ITEMS];   // their indices in order, after the keys have been read
    };
    uint32_t base[THREADS * ITEMS + 4];
    uint32_t red[2][THREADS / kWave];
    uint32_t tmp[THREADS / kWave];
    uint32_t most[THREADS / kWave];
};

template <int THREADS>
__device__ __forceinline__ void group_sync() {
    if (THREADS == kWave)
        wave_lds_order();
    else
        __syncthreads();
}

// Smallest and largest x over the group, in every thread. Contains group_sync.
template <int THREADS>
__device__ __forceinline__ void group_range(uint32_t& lo, uint32_t& hi, uint32_t (*red)[THREADS / kWave]) {
    constexpr int kW = THREADS / kWave;
    lo = ~wave_max(~lo);
    hi = wave_max(hi);
    if (kW == 1) return;
    if (lane_id() == 0) {
        red[0][threadIdx.x >> 6] = lo;
        red[1][threadIdx.x >> 6] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kW; ++q) {
        lo = min(lo, red[0][q]);
        hi = max(hi, red[1][q]);
    }
}

// Exclusive scan of x over the group's threads. Contains group_sync.
template <int THREADS>
__device__ __forceinline__ uint32_t group_exclusive_scan(uint32_t x, uint32_t* tmp) {
    uint32_t incl = wave_inclusive_scan(x);
    if (THREADS > kWave) {
        const uint32_t w = threadIdx.x >> 6;
        if (lane_id() == kWave - 1) tmp[w] = incl;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < THREADS / kWave; ++q) incl += (uint32_t)q < w ? tmp[q] : 0u;
    }
    return incl - x;
}

// The piece's keys as its threads hold them: item i of thread t is entry i * THREADS + t.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void load_piece(const SortSource& src, uint32_t start, uint32_t n,
                                           const uint32_t* pidx, uint64_t (&k)[ITEMS]) {
    const uint32_t t = threadIdx.x % THREADS;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) k[i] = src.at(start + min((uint32_t)i * THREADS + t, n - 1u), pidx);
}

template <int THREADS, int ITEMS>
__device__ __forceinline__ void sort_piece(SortShared<THREADS, ITEMS>& sh, uint64_t (&k)[ITEMS], uint32_t start,
                                           uint32_t n, uint32_t tile, uint32_t* pidx, uint64_t* __restrict__ keys64) {
    constexpr int kW = THREADS / kWave;
    constexpr uint32_t kCap = THREADS * ITEMS;
    static_assert(ITEMS % 4 == 0, "whole 16-byte vectors of buckets per thread");
    const uint32_t t = threadIdx.x % THREADS, w = t >> 6, l = lane_id();
    uint32_t lo_z = ~0u, hi_z = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {   // (past the end: the last entry again)
        lo_z = min(lo_z, (uint32_t)(k[i] >> 32));
        hi_z = max(hi_z, (uint32_t)(k[i] >> 32));
    }
#pragma unroll
    for (int i = 0; i < ITEMS; i += 4) *reinterpret_cast<uint4*>(&sh.base[i * THREADS + 4 * t]) = make_uint4(0u, 0u, 0u, 0u);
    *reinterpret_cast<uint4*>(&sh.part[4 * t]) = make_uint4(0u, 0u, 0u, 0u);
    group_range<THREADS>(lo_z, hi_z, sh.red);
    const bool equal = lo_z == hi_z;   // uniform over the group
    if (equal) {
        lo_z = ~0u;
        hi_z = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            lo_z = min(lo_z, (uint32_t)k[i]);
            hi_z = max(hi_z, (uint32_t)k[i]);
        }
        group_sync<THREADS>();
        group_range<THREADS>(lo_z, hi_z, sh.red);
    }
    group_sync<THREADS>();
    const BucketMap map(lo_z, hi_z, equal, 4 * THREADS);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if ((uint32_t)i * THREADS + t < n) atomicAdd(&sh.part[map.of(k[i])], 1u);
    group_sync<THREADS>();
    {
        const uint4 q = *reinterpret_cast<const uint4*>(&sh.part[4 * t]);
        const uint32_t e = group_exclusive_scan<THREADS>(q.x + q.y + q.z + q.w, sh.tmp);
        *reinterpret_cast<uint4*>(&sh.part[4 * t]) = make_uint4(e, e + q.x, e + q.x + q.y, e + q.x + q.y + q.z);
        if (t == THREADS - 1) sh.part[4 * THREADS] = n;
    }
    group_sync<THREADS>();
    uint32_t slot[ITEMS];   // bucket, and the arrival in it
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const float at = map.at(k[i]);
        const uint32_t p = map.bucket(at), b0 = sh.part[p], c = max(sh.part[p + 1] - b0, 1u);
        const uint32_t b = b0 + min((uint32_t)((at - (float)p) * (float)c), c - 1u);
        slot[i] = (uint32_t)i * THREADS + t < n ? atomicAdd(&sh.base[b], 1u) << 16 | b : b;
    }
    group_sync<THREADS>();
    // exclusive scan of ITEMS consecutive buckets per thread, and the largest bucket
    uint32_t c[ITEMS], most = 0, sum = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; i += 4) {
        const uint4 q = *reinterpret_cast<const uint4*>(&sh.base[ITEMS * t + i]);
        c[i] = q.x;
        c[i + 1] = q.y;
        c[i + 2] = q.z;
        c[i + 3] = q.w;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        most = max(most, c[i]);
        sum += c[i];
    }
    most = wave_max(most);
    if (kW > 1 && l == 0) sh.most[w] = most;
    uint32_t e = group_exclusive_scan<THREADS>(sum, sh.tmp);
    if (kW > 1) {
#pragma unroll
        for (int q = 0; q < kW; ++q) most = max(most, sh.most[q]);
    }
#pragma unroll
    for (int i = 0; i < ITEMS; i += 4) {
        const uint32_t e1 = e + c[i], e2 = e1 + c[i + 1], e3 = e2 + c[i + 2];
        *reinterpret_cast<uint4*>(&sh.base[ITEMS * t + i]) = make_uint4(e, e1, e2, e3);
        e = e3 + c[i + 3];
    }
    if (t == THREADS - 1) sh.base[kCap] = n;
    group_sync<THREADS>();
    uint32_t lo[ITEMS], len[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t b = slot[i] & 0xFFFFu;
        lo[i] = sh.base[b];
        len[i] = (uint32_t)i * THREADS + t < n ? sh.base[b + 1] - lo[i] : 0u;
        if (len[i]) sh.key[lo[i] + (slot[i] >> 16)] = k[i];
    }
    group_sync<THREADS>();
    if (most <= kBucketMax) {
        // the ITEMS buckets side by side, so that their reads are in flight together
        uint32_t rank[ITEMS], longest = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            rank[i] = 0;
            longest = max(longest, len[i]);
        }
        if (longest > 1u) {
            for (uint32_t q = 0; q < longest; ++q) {
                uint64_t x[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) x[i] = sh.key[lo[i] + min(q, max(len[i], 1u) - 1u)];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) rank[i] += q < len[i] && x[i] < k[i] ? 1u : 0u;
            }
        }
        group_sync<THREADS>();   // every key has been read
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (!len[i]) continue;
            sh.sorted[lo[i] + rank[i]] = (uint32_t)k[i];
            if (keys64) keys64[start + lo[i] + rank[i]] = (uint64_t)tile << 32 | k[i] >> 32;
        }
        group_sync<THREADS>();
    } else {
        uint32_t size = 2;
        while (size < n) size <<= 1;   // at most kCap, uniform
        for (uint32_t p = n + t; p < size; p += THREADS) sh.key[p] = ~0ull;
        group_sync<THREADS>();
        for (uint32_t s = 2; s <= size; s <<= 1) {
            for (uint32_t d = s >> 1; d > 0; d >>= 1) {
                for (uint32_t p = t; p < size / 2; p += THREADS) {
                    const uint32_t a = 2 * (p & ~(d - 1u)) | (p & (d - 1u)), c2 = a | d;
                    const uint64_t x = sh.key[a], y = sh.key[c2];
                    if ((x > y) == ((a & s) == 0u)) {
                        sh.key[a] = y;
                        sh.key[c2] = x;
                    }
                }
                group_sync<THREADS>();
            }
        }
        uint64_t r[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) r[i] = sh.key[min((uint32_t)i * THREADS + t, n - 1u)];
        group_sync<THREADS>();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t p = (uint32_t)i * THREADS + t;
            if (p >= n) continue;
            sh.sorted[p] = (uint32_t)r[i];
            if (keys64) keys64[start + p] = (uint64_t)tile << 32 | r[i] >> 32;
        }
        group_sync<THREADS>();
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t p = (uint32_t)i * THREADS + t;
        if (p < n) pidx[start + p] = sh.sorted[p];
    }
}

// Up to 64 entries by one wave, one per lane: the rank is the number of smaller keys.
__device__ __forceinline__ void sort_lanes(const SortSource& src, uint32_t start, uint32_t n, uint32_t tile,
                                           uint32_t* __restrict__ pidx, uint64_t* __restrict__ keys64) {
    const uint32_t l = lane_id();
    const uint64_t key = src.at(start + min(l, n - 1u), pidx);
    uint32_t rank = 0;
    for (uint32_t j = 0; j < n; ++j) {
        const uint64_t kj = (uint64_t)__builtin_amdgcn_readlane((uint32_t)(key >> 32), (int)j) << 32 |
                            __builtin_amdgcn_readlane((uint32_t)key, (int)j);
        rank += kj < key ? 1u : 0u;
    }
    if (l >= n) return;
    pidx[start + rank] = (uint32_t)key;
    if (keys64) keys64[start + rank] = (uint64_t)tile << 32 | key >> 32;
}

// Item i of a size class: the pieces of step 5, then the listed tiles; none past the end.
__device__ __forceinline__ SortItem class_item(const SortItem* __restrict__ items, uint32_t m,
                                               const uint32_t* __restrict__ tiles, uint32_t total,
                                               const uint32_t* __restrict__ ranges, uint32_t i) {
    SortItem it{0, 0, 0, 0};
    if (i >= total) return it;
    if (i < m) return items[i];
    it.tile = tiles[i - m];
    it.start = ranges[2 * (size_t)it.tile];
    it.n = ranges[2 * (size_t)it.tile + 1] - it.start;
    return it;
}

// The workgroup's share of a size class; the next item is fetched while the current one is
// sorted.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void sort_class(SortShared<THREADS, ITEMS>& sh, const BinArrays& A,
                                           const SortItem* __restrict__ items, uint32_t m,
                                           const uint32_t* __restrict__ tiles, uint32_t total, uint32_t block,
                                           uint32_t blocks, const uint32_t* __restrict__ ranges, uint32_t* pidx,
                                           uint64_t* __restrict__ keys64) {
    SortItem cur = class_item(items, m, tiles, total, ranges, block);
    while (cur.n) {   // uniform
        block += blocks;
        const SortItem next = class_item(items, m, tiles, total, ranges, block);
        uint64_t k[ITEMS];
        load_piece<THREADS, ITEMS>(SortSource{A.key, A.z_alt, cur.buf}, cur.start, cur.n, pidx, k);
        sort_piece<THREADS, ITEMS>(sh, k, cur.start, cur.n, cur.tile, pidx, keys64);
        __syncthreads();
        cur = next;
    }
}

// Step 6, segments and pieces of 1025 to 4096 entries.
constexpr int kBigThreads = 1024;
__global__ void __launch_bounds__(kBigThreads) __attribute__((amdgpu_waves_per_eu(8))) bin_sort_big_kernel(const BinArrays A,
                                                                   const uint32_t* __restrict__ ranges, uint32_t* pidx,
                                                                   uint64_t* __restrict__ keys64,
                                                                   const int32_t* __restrict__ status) {
    __shared__ SortShared<kBigThreads, 4> sh;
    if (*status != kStatusOk) return;
    const uint32_t n = min(A.counters[kNumBig], A.list_max), m = min(A.counters[kNumBigItems], A.item_max);
    sort_class<kBigThreads, 4>(sh, A, A.big_item, m, A.big, n + m, blockIdx.x, gridDim.x, ranges, pidx, keys64);
}

// Step 6, the others: the first workgroups take the listed segments and pieces of up to 1024
// entries, the rest one tile of up to 256 entries per wave.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) bin_sort_mid_kernel(const BinArrays A, uint32_t mid_blocks, uint32_t tiles,
                                                           const uint32_t* __restrict__ ranges, uint32_t* pidx,
                                                           uint64_t* __restrict__ keys64,
                                                           const int32_t* __restrict__ status) {
    __shared__ union {
        SortShared<256, 4> mid;
        SortShared<kWave, 4> small[4];
    } sh;
    if (*status != kStatusOk) return;
    if (blockIdx.x >= mid_blocks) {
        const uint32_t b = blockIdx.x - mid_blocks, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t tile = 4 * xcd_swizzle(b, gridDim.x - mid_blocks) + w;
        if (tile >= tiles) return;
        const uint32_t start = ranges[2 * (size_t)tile], n = ranges[2 * (size_t)tile + 1] - start;
        if (n == 0 || n > kSmallMax) return;
        const SortSource src{A.key, A.z_alt, 0u};
        if (n <= (uint32_t)kWave) {
            sort_lanes(src, start, n, tile, pidx, keys64);
        } else {
            uint64_t k[4];
            load_piece<kWave, 4>(src, start, n, pidx, k);
            sort_piece<kWave, 4>(sh.small[w], k, start, n, tile, pidx, keys64);
        }
        return;
    }
    const uint32_t n = min(A.counters[kNumMid], A.list_max), m = min(A.counters[kNumMidItems], A.item_max);
    sort_class<256, 4>(sh.mid, A, A.mid_item, m, A.mid, n + m, blockIdx.x, mid_blocks, ranges, pidx, keys64);
}

// ---- Step 5: long segments ----------------------------------------------------------------------

// A workgroup takes a segment of more than kBigMax entries (from a device-wide counter) and
// distributes it over 4096 buckets of its depth range, from one buffer to the other;
// consecutive buckets whose entries start in the same 2048 make one piece (at most 4095
// entries), a bucket of more than 2048 entries is a piece of its own, and pieces longer than
// kBigMax are distributed again (the range of a bucket is at most a 4096th of its parent's, and
// equal depths are told apart by their indices, so this ends after a few levels). A level
// reads the keys for their range, for the buckets' counts and for the distribution, and
// writes them once; four radix passes over 4096-entry chunks wrote them four times and took
// thirteen launches, whether or not a tile needed them.
constexpr uint32_t kParts = 4096;
constexpr uint32_t kPartGroup = 2048;
// The distributed entries go through LDS, kPartStage at a time, so that they are written in order:
// scattered 4-byte writes left L2 as partial lines and took about 14 cycles of a CU per entry. A
// segment of up to kMaxWindows times as many is read again for each window of pieces; each
// further window reads the whole segment, so a longer one is scattered directly. Ten 1080p
// views 41 -> 27 us, one 18 -> 12.5, three views of a serving batch 40 -> 27, eight 4K views
// 850 -> 772 us (1 window: 836, 2: 792, 8: 769, 32: 1002).
constexpr uint32_t kPartStage = 14720;   // one workgroup's LDS of a CU with the rest
constexpr uint32_t kMaxWindows = 4;
constexpr uint32_t kPartLoads = 8;       // loads in flight per thread

struct __align__(16) PartShared {
    uint32_t base[kParts];
    uint32_t first[kParts + 1];   // start of each piece
    uint16_t bucket[kParts];      // its first bucket
    uint32_t red[2][kBinWaves];
    uint32_t tmp[kBinWaves];
    uint32_t last[kBinWaves];
    uint32_t item, depth, n_mid, n_big, at_mid, at_big, cur[3];
    __align__(16) uint64_t stage[kPartStage];   // the distributed entries of a segment of at most as many
};

__global__ void __launch_bounds__(kBinThreads) bin_partition_kernel(const BinArrays A, uint32_t* pidx,
                                                                    const int32_t* __restrict__ status) {
    __shared__ PartShared sh;
    if (*status != kStatusOk) return;
    const uint32_t t = threadIdx.x, w = t >> 6, l = lane_id();
    const uint32_t n_large = min(A.counters[kNumLarge], A.large_max);
    for (;;) {
        __syncthreads();
        if (t == 0) sh.item = atomicAdd(&A.counters[kWork], 1u);
        __syncthreads();
        if (sh.item >= n_large) break;   // uniform
        const SortItem seg = A.large[sh.item];
        uint2* stack = A.stack + seg.start / kBigMax;
        uint32_t start = seg.start, n = seg.n, buf = 0;
        if (t == 0) sh.depth = 0;
        for (;;) {
            const SortSource src{A.key, A.z_alt, buf};
            // the range of the depths, and where they are all equal of the indices
            uint32_t lo = ~0u, hi = 0, lo_i = ~0u, hi_i = 0;
            for (uint32_t p0 = t; p0 < n; p0 += kPartLoads * kBinThreads) {
                uint64_t k[kPartLoads];
#pragma unroll
                for (uint32_t i = 0; i < kPartLoads; ++i)
                    k[i] = src.at(start + min(p0 + i * kBinThreads, n - 1u), pidx);
#pragma unroll
                for (uint32_t i = 0; i < kPartLoads; ++i) {
                    lo = min(lo, (uint32_t)(k[i] >> 32));
                    hi = max(hi, (uint32_t)(k[i] >> 32));
                    lo_i = min(lo_i, (uint32_t)k[i]);
                    hi_i = max(hi_i, (uint32_t)k[i]);
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < kParts / kBinThreads; ++q) sh.base[q * kBinThreads + t] = 0u;
            if (t == 0) sh.n_mid = sh.n_big = 0;
            group_range<kBinThreads>(lo, hi, sh.red);
            const bool equal = lo == hi;
            __syncthreads();
            if (equal) {
                lo = lo_i;
                hi = hi_i;
                group_range<kBinThreads>(lo, hi, sh.red);
                __syncthreads();
            }
            const BucketMap map(lo, hi, equal, kParts);
            for (uint32_t p0 = t; p0 < n; p0 += kPartLoads * kBinThreads) {
                uint64_t k[kPartLoads];
#pragma unroll
                for (uint32_t i = 0; i < kPartLoads; ++i)
                    k[i] = src.at(start + min(p0 + i * kBinThreads, n - 1u), pidx);
#pragma unroll
                for (uint32_t i = 0; i < kPartLoads; ++i)
                    if (p0 + i * kBinThreads < n) atomicAdd(&sh.base[map.of(k[i])], 1u);
            }
            __syncthreads();
            // four consecutive buckets per thread: bases, and which of them start a piece
            static_assert(kParts == 4 * kBinThreads, "four buckets per thread");
            const uint4 c4 = *reinterpret_cast<const uint4*>(&sh.base[4 * t]);
            const uint32_t c[4] = {c4.x, c4.y, c4.z, c4.w};
            uint32_t total;
            uint32_t e = block_exclusive_scan<kBinWaves, uint32_t>(c4.x + c4.y + c4.z + c4.w, sh.tmp, total);
            uint32_t at[4], tag = 0;   // tag: the last non-empty bucket so far, 2 (group + 1) + alone
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                at[q] = e;
                e += c[q];
                if (c[q]) tag = 2u * (at[q] / kPartGroup + 1u) + (c[q] > kPartGroup ? 1u : 0u);
            }
            const uint64_t has = ballot64(tag != 0u);
            const uint64_t below = has & ((1ull << l) - 1ull);
            if (l == 0) sh.last[w] = has ? (uint32_t)__builtin_amdgcn_readlane(tag, 63 - __builtin_clzll(has)) : 0u;
            uint32_t prev = __shfl(tag, below ? 63 - __clzll((long long)below) : 0, kWave);
            __syncthreads();
            if (!below) {
                prev = 0;
                for (int q = (int)w - 1; q >= 0 && !prev; --q) prev = sh.last[q];
            }
            bool starts[4];
            uint32_t ns = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                starts[q] = false;
                if (!c[q]) continue;
                const uint32_t now = 2u * (at[q] / kPartGroup + 1u) + (c[q] > kPartGroup ? 1u : 0u);
                starts[q] = now != prev || (now & 1u);
                prev = now;
                ns += starts[q] ? 1u : 0u;
            }
            uint32_t pieces;
            uint32_t s = block_exclusive_scan<kBinWaves, uint32_t>(ns, sh.tmp, pieces);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                sh.base[4 * t + q] = at[q];
                if (!starts[q]) continue;
                sh.bucket[s] = (uint16_t)(4 * t + q);
                sh.first[s++] = at[q];
            }
            if (t == 0) sh.first[pieces] = n;
            __syncthreads();
            auto put = [&](uint32_t d, uint64_t k) {
                if (buf) {
                    A.key[d] = k;
                } else {
                    A.z_alt[d] = (uint32_t)(k >> 32);
                    pidx[d] = (uint32_t)k;
                }
            };
            // window by window: the pieces [i0, i1) of buckets [b0, b1) and positions [w0, w1)
            const bool windows = n <= kMaxWindows * kPartStage;   // uniform
            for (uint32_t i0 = 0; i0 < pieces;) {
                const uint32_t w0 = windows ? sh.first[i0] : 0u, b0 = windows ? sh.bucket[i0] : 0u;
                uint32_t i1 = windows ? i0 + 1u : pieces;
                while (i1 < pieces && sh.first[i1 + 1] - w0 <= kPartStage) ++i1;
                const uint32_t w1 = sh.first[i1], nb = (i1 < pieces ? sh.bucket[i1] : kParts) - b0;
                const bool staged = w1 - w0 <= kPartStage;
                for (uint32_t p0 = t; p0 < n; p0 += kPartLoads * kBinThreads) {
                    uint64_t k[kPartLoads];
#pragma unroll
                    for (uint32_t i = 0; i < kPartLoads; ++i)
                        k[i] = src.at(start + min(p0 + i * kBinThreads, n - 1u), pidx);
#pragma unroll
                    for (uint32_t i = 0; i < kPartLoads; ++i) {
                        const uint32_t b = map.of(k[i]);
                        if (p0 + i * kBinThreads >= n || b - b0 >= nb) continue;
                        const uint32_t d = atomicAdd(&sh.base[b], 1u);
                        if (staged)
                            sh.stage[d - w0] = k[i];
                        else
                            put(start + d, k[i]);
                    }
                }
                if (staged) {
                    __syncthreads();
                    for (uint32_t p = w0 + t; p < w1; p += kBinThreads) put(start + p, sh.stage[p - w0]);
                    __syncthreads();   // the window has been read
                }
                i0 = i1;
            }
            // the pieces: listed for step 6, or pending
            const uint32_t to = buf ^ 1u;
            for (uint32_t q0 = 0; q0 < pieces; q0 += kBinThreads) {
                const uint32_t q = q0 + t;
                const uint32_t f = q < pieces ? sh.first[q] : 0u, pn = q < pieces ? sh.first[q + 1] - f : 0u;
                uint32_t i = 0;
                if (pn > kBigMax)
                    stack[atomicAdd(&sh.depth, 1u)] = make_uint2(start + f, pn | to << 31);
                else if (pn)
                    i = atomicAdd(pn <= kMidMax ? &sh.n_mid : &sh.n_big, 1u);
                __syncthreads();
                if (t == 0) {
                    sh.at_mid = sh.n_mid ? atomicAdd(&A.counters[kNumMidItems], sh.n_mid) : 0u;
                    sh.at_big = sh.n_big ? atomicAdd(&A.counters[kNumBigItems], sh.n_big) : 0u;
                }
                __syncthreads();
                if (pn && pn <= kBigMax) {
                    const bool mid = pn <= kMidMax;
                    i += mid ? sh.at_mid : sh.at_big;
                    if (i < A.item_max) (mid ? A.mid_item : A.big_item)[i] = SortItem{start + f, pn, seg.tile, to};
                }
                __syncthreads();
                if (t == 0) sh.n_mid = sh.n_big = 0;
                __syncthreads();
            }
            // the next pending range (written by this workgroup before the barriers above)
            if (t == 0) {
                sh.cur[1] = 0;
                if (sh.depth) {
                    const uint2 r = stack[--sh.depth];
                    sh.cur[0] = r.x;
                    sh.cur[1] = r.y & 0x7FFFFFFFu;
                    sh.cur[2] = r.y >> 31;
                }
            }
            __syncthreads();
            start = sh.cur[0];
            n = sh.cur[1];
            buf = sh.cur[2];
            __syncthreads();
            if (!n) break;   // uniform
        }
    }
}

// ---- Host -----------------------------------------------------------------------------------------

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static uint32_t view_tiles(const isogs_camera& c) {
    return (uint32_t)((c.width + kTile - 1) / kTile) * (uint32_t)((c.height + kTile - 1) / kTile);
}

// The chunking of a call: particles per chunk. Two workgroups of 1024 threads fit a CU (one with
// the larger band), so the chunks of all views together are at most what runs at once: 512, or
// 256 where fewer particles are worth less than the matrix rows (4 bytes per tile of the view)
// that more chunks cost. With 256 and 512, 1080p views of 1M particles: one 97 and 104 us, three 186
// and 195, four 291 and 283, six 366 and 362, ten 623 and 614. Every band of a view takes each
// chunk, so a view of several bands has that many times fewer chunks (twice those 256 workgroups
// above four bands, whose shares of the particles differ more): the matrix then has at most 256
// kBandLarge counts (512 above four bands), 38 MB (75 MB), and a row per view, however many tiles.
// With 256 and 512 workgroups: 5120 x 2880 of 1M particles (two bands) 190 and 220 us, 12288 x 6912 of
// 300k (nine) 451 and 423, 16384 x 16384 of 1M (29) 1.96 and 1.80 ms.
static uint32_t chunk_particles(uint64_t n_total, int32_t nv, bool large_band, uint32_t bands) {
    const uint32_t least = n_total <= kGroupMaxParticles ? 128u : 1024u;
    const uint32_t target = bands > 4                         ? std::max(kMaxChunks / bands, 1u)
                            : large_band || n_total < 4000000 ? kMaxChunks / 2 / bands
                                                              : kMaxChunks;
    const uint32_t rows = std::max(target - std::min<uint32_t>((uint32_t)nv, target / 2), 1u);
    return (uint32_t)std::max<uint64_t>(least, (n_total + rows - 1) / rows);
}

BinSortPlan plan_bin_sort(const int32_t* n_per_view, const isogs_camera* cams, int32_t nv, uint64_t capacity,
                          size_t limit) {
    BinSortPlan p{};
    p.capacity = capacity;
    uint64_t n = 0, tiles = 0;
    uint32_t most_tiles = 0;
    for (int v = 0; v < nv; ++v) {
        n += (uint64_t)n_per_view[v];
        tiles += view_tiles(cams[v]);
        most_tiles = std::max(most_tiles, view_tiles(cams[v]));
    }
    p.n_total = (uint32_t)n;
    p.tiles_total = (uint32_t)tiles;
    p.large_band = most_tiles > kBandSmall;
    p.bands = p.large_band ? (most_tiles + kBandLarge - 1) / kBandLarge : 1u;
    // The size that callers are told: 20 bytes per entry of capacity and tile, a tile digit
    // histogram per 4096 entries and the tables of the long segments. The layout below takes
    // more for scenes of many more particles than entries (the boxes) and for few entries in
    // many tiles (the matrix); a caller whose workspace cannot grow (`limit`) then gets a layout
    // without the packed boxes (step 4 reads the records again), and where that is not enough
    // with half the chunks, as often as it takes: at one per view it never takes more.
    const uint64_t sort_tiles = (capacity + 4095) / 4096, long_max = std::min<uint64_t>(tiles, capacity / 16385 + 1);
    const size_t told = 5 * align256(capacity * 4) + (size_t)sort_tiles * 2048 + (size_t)(sort_tiles + long_max) * 1028 +
                        (size_t)long_max * 40 + (size_t)tiles * 20 + (n + 2047) / 2048 * 4 + 40960;
    p.per = chunk_particles(n, nv, p.large_band, p.bands);
    for (int small = 0;; ++small) {
        if (small > 1) p.per = (uint32_t)std::min<uint64_t>(2ull * p.per, 0x7FFFFFFFu);
        uint64_t chunks = 0, blocks = 0, m = 0;
        for (int v = 0; v < nv; ++v) {
            const uint64_t c = ((uint64_t)n_per_view[v] + p.per - 1) / p.per, vt = view_tiles(cams[v]);
            chunks += c;
            blocks += (vt + 1 + kColTiles - 1) / kColTiles;
            m += c * (vt + 1);
        }
        p.chunks = (uint32_t)chunks;
        p.blocks = (uint32_t)blocks;
        p.list_max = (uint32_t)std::min<uint64_t>(tiles, capacity / kSmallMax + 1);
        p.large_max = (uint32_t)std::min<uint64_t>(tiles, capacity / kBigMax + 1);
        // pieces of step 5: at most six per 4096 entries of a level and one more, a few levels
        p.item_max = (uint32_t)(64 * (capacity / kBigMax + 1));
        size_t off = 0;
        auto take = [&off](size_t bytes) {
            const size_t at = off;
            off = align256(off + bytes);
            return at;
        };
        p.off_key = take(capacity * 8);
        p.off_z = take(capacity * 4);
        p.off_box = take(small ? 0 : n * 8);
        p.boxes = !small;
        p.off_m = take(m * 4);
        p.off_tile_pre = take(tiles * 4);
        p.off_tile_tot = take(tiles * 4);
        p.off_missing = take((size_t)nv * 8);
        p.off_block_sum = take(blocks * 4);
        p.off_chunk_sum = take(chunks * 8);
        p.off_miss = take(p.bands > 1 ? (size_t)chunks * p.bands * 4 : 0);
        p.off_counters = take(kCounterWords * 4);
        p.off_lists = take((size_t)p.list_max * 8 + (size_t)p.large_max * sizeof(SortItem) + 16);
        p.off_items = take((size_t)p.item_max * 2 * sizeof(SortItem));
        p.off_stack = take((capacity / kBigMax + 2) * 8);
        p.bytes = std::max(off, told);
        if (p.bytes <= limit || told > limit || (small && p.per >= n)) break;
    }
    return p;
}

int launch_bin_sort(const BinSortPlan& plan, const isogs_projected* proj, const int32_t* n_per_view,
                    const isogs_camera* cams, int32_t nv, const isogs_bins* bins, void* ws, hipStream_t stream) {
    char* base = static_cast<char*>(ws);
    auto at = [base](size_t off) { return reinterpret_cast<uint32_t*>(base + off); };
    BinArrays A{};
    A.key = reinterpret_cast<uint64_t*>(base + plan.off_key);
    A.z_alt = at(plan.off_z);
    A.box = plan.boxes ? reinterpret_cast<uint2*>(base + plan.off_box) : nullptr;
    A.m = at(plan.off_m);
    A.tile_pre = at(plan.off_tile_pre);
    A.tile_tot = at(plan.off_tile_tot);
    A.missing = at(plan.off_missing);
    A.missing_at = A.missing + nv;
    A.block_sum = at(plan.off_block_sum);
    A.chunk_sum = reinterpret_cast<uint64_t*>(base + plan.off_chunk_sum);
    A.counters = at(plan.off_counters);
    A.large = reinterpret_cast<SortItem*>(base + plan.off_lists);
    A.mid = reinterpret_cast<uint32_t*>(A.large + plan.large_max);
    A.big = A.mid + plan.list_max;
    A.mid_item = reinterpret_cast<SortItem*>(base + plan.off_items);
    A.big_item = A.mid_item + plan.item_max;
    A.stack = reinterpret_cast<uint2*>(base + plan.off_stack);
    A.list_max = plan.list_max;
    A.large_max = plan.large_max;
    A.item_max = plan.item_max;
    A.blocks = plan.blocks;
    A.chunks = plan.chunks;
    A.views = (uint32_t)nv;
    const float4* record = reinterpret_cast<const float4*>(proj->record);
    // eight lanes per particle: few particles, or (a view of several bands) boxes of many tiles,
    // told by a capacity of 16 entries per particle: 300k particles with 50 each in 16384 x 16384
    // take 1.28 ms with eight lanes and 1.65 with one, 6M with 10 each 4.17 and 3.33
    const bool group = plan.n_total <= kGroupMaxParticles || (plan.bands > 1 && plan.capacity >= 16ull * plan.n_total);
    const uint32_t band = plan.large_band ? kBandLarge : kBandSmall;

    // groups of up to kMaxViews views: counts and columns, then (all views) the scans, then
    // placement
    int32_t most = 0;
    for (int stage = 0; stage < 2; ++stage) {
        uint32_t p_off = 0, tile_base = 0, chunk0 = 0, block0 = 0;
        uint64_t m_off = 0;
        for (int v0 = 0; v0 < nv; v0 += kMaxViews) {
            BinPack pk{};
            pk.nv = min(kMaxViews, nv - v0);
            pk.view0 = (uint32_t)v0;
            pk.tile0 = tile_base;
            uint32_t chunks = 0, blocks = 0, bands = 1;
            for (int j = 0; j < pk.nv; ++j) {
                const isogs_camera& cam = cams[v0 + j];
                BinView& d = pk.v[j];
                d.p_off = p_off;
                d.n = (uint32_t)n_per_view[v0 + j];
                d.tile_base = tile_base;
                d.width = cam.width;
                d.height = cam.height;
                d.tiles_x = (cam.width + kTile - 1) / kTile;
                d.tiles_y = (cam.height + kTile - 1) / kTile;
                d.tiles = view_tiles(cam);
                d.per = plan.per;
                d.chunks = (uint32_t)(((uint64_t)d.n + plan.per - 1) / plan.per);
                d.chunk0 = chunk0;
                d.block0 = block0;
                d.m_off = m_off;
                pk.chunk_begin[j] = chunks;
                pk.block_begin[j] = blocks;
                chunks += d.chunks;
                blocks += (d.tiles + 1 + kColTiles - 1) / kColTiles;
                bands = std::max(bands, (d.tiles + band - 1) / band);
                most = std::max(most, n_per_view[v0 + j]);
                p_off += d.n;
                tile_base += d.tiles;
                chunk0 += d.chunks;
                block0 += (d.tiles + 1 + kColTiles - 1) / kColTiles;
                m_off += (uint64_t)d.chunks * (d.tiles + 1);
            }
            pk.chunk_begin[pk.nv] = chunks;
            pk.block_begin[pk.nv] = blocks;
            pk.tiles = tile_base - pk.tile0;
            pk.bands = bands;
            pk.miss_pitch = plan.bands;
            pk.miss = at(plan.off_miss);
            if (stage == 0) {
                auto count = plan.bands > 1
                                 ? (group ? bin_count_kernel<kBandLarge, 8, true> : bin_count_kernel<kBandLarge, 1, true>)
                             : plan.large_band
                                 ? (group ? bin_count_kernel<kBandLarge, 8, false> : bin_count_kernel<kBandLarge, 1, false>)
                                 : (group ? bin_count_kernel<kBandSmall, 8, false> : bin_count_kernel<kBandSmall, 1, false>);
                if (chunks)
                    hipLaunchKernelGGL(count, dim3(work_blocks(chunks, bands)), dim3(kBinThreads), 0, stream, pk, record,
                                       proj->tile_count, A);
                auto columns = plan.bands > 1 ? bin_columns_kernel<true> : bin_columns_kernel<false>;
                hipLaunchKernelGGL(columns, dim3(blocks), dim3(kBinThreads), 0, stream, pk, A);
            } else {
                auto place = plan.bands > 1
                                 ? (group ? bin_place_kernel<kBandLarge, 8, true> : bin_place_kernel<kBandLarge, 1, true>)
                             : plan.large_band
                                 ? (group ? bin_place_kernel<kBandLarge, 8, false> : bin_place_kernel<kBandLarge, 1, false>)
                                 : (group ? bin_place_kernel<kBandSmall, 8, false> : bin_place_kernel<kBandSmall, 1, false>);
                hipLaunchKernelGGL(place, dim3(work_blocks(chunks, bands) + (pk.tiles + kBinThreads - 1) / kBinThreads),
                                   dim3(kBinThreads), 0, stream, pk, record, proj->depth, proj->tile_count, A,
                                   bins->status, bins->count, bins->ranges, bins->offsets, bins->pidx);
            }
        }
        if (stage == 0)
            hipLaunchKernelGGL(bin_top_kernel, dim3(1), dim3(kBinThreads), 0, stream, A, plan.capacity, bins->count,
                               bins->status);
        if (hipPeekAtLastError() != hipSuccess) return -1;
    }
    if (plan.capacity == 0) return 0;
    // a tile's list holds each particle of its view at most once: without a view of more
    // particles than a length there is no such segment, and nothing is launched for it
    if ((uint32_t)most > kBigMax) {
        const unsigned grid = std::min<unsigned>(plan.large_max, 512u);
        hipLaunchKernelGGL(bin_partition_kernel, dim3(grid), dim3(kBinThreads), 0, stream, A, bins->pidx, bins->status);
    }
    if ((uint32_t)most > kMidMax) {
        const unsigned grid = std::min<unsigned>(plan.list_max + plan.item_max, 768u);
        hipLaunchKernelGGL(bin_sort_big_kernel, dim3(grid), dim3(kBigThreads), 0, stream, A, bins->ranges, bins->pidx,
                           bins->keys, bins->status);
    }
    const uint32_t mid_blocks = (uint32_t)most > kSmallMax ? std::min<uint32_t>(plan.list_max + plan.item_max, 2048u) : 0u;
    hipLaunchKernelGGL(bin_sort_mid_kernel, dim3(mid_blocks + (plan.tiles_total + 3) / 4), dim3(256), 0, stream, A,
                       mid_blocks, plan.tiles_total, bins->ranges, bins->pidx, bins->keys, bins->status);
    return hipPeekAtLastError() == hipSuccess ? 0 : -1;
}

}  // namespace isogs
