// Tile-raster helpers shared by the forward and backward compositing kernels.
#pragma once

#include "common.h"
#include "kernels.h"

namespace isogs {

constexpr int kBatch = 256;   // forward: entries staged in LDS per round (one per thread)

// Compositing checkpoints: at every kCkptChunk-th position of a long tile list (a multiple
// of the forward batch) the forward can store each pixel's {T, r, g, b} before that entry,
// so that the backward can walk the chunks of the list on different workgroups. The
// checkpoints of the tile whose list starts at global entry `start` occupy slots
// start / kCkptChunk + k (k >= 1), which never overlap between tiles; a slot holds one
// float4 per pixel (thread) of the tile. Lists of at least kChunkedMin entries (length
// class kChunkedClass and up, the class being the bit length) are the long ones.
constexpr uint32_t kCkptChunk = 256;
constexpr uint32_t kChunkedMin = 2 * kCkptChunk;
constexpr int kChunkedClass = 10;
static_assert(kCkptChunk % 256 == 0, "checkpoints sit on forward batch boundaries");
static_assert(kCkptChunk == ISOGS_CKPT_CHUNK, "the header states the checkpoint spacing");
static_assert((1u << (kChunkedClass - 1)) == kChunkedMin, "class of the shortest chunked list");

__host__ __device__ inline uint32_t ckpt_slot(uint32_t start, uint32_t k) { return start / kCkptChunk + k; }
__host__ __device__ inline bool chunked_list(uint32_t len) { return len >= kChunkedMin; }

// Longest-list-first tile queues: list length classes 0, then 32 - clz(length); a queue
// starts with its class histogram (kBuckets words).
constexpr int kBuckets = 33;
constexpr int kDummy = kBatch; // staged slot of a zero-opacity record that pads the lists

// Queue position that block b of nb takes: consecutive blocks run on different XCDs, so of
// each 8 kQueueRun positions an XCD takes kQueueRun consecutive ones, mostly neighbouring tiles,
// which share records in its L2. Ten views of 1080p forward: 618 us with runs of 1, 574 with 8,
// 581 with 32, 622 with 128 (the longest lists then crowd on one XCD).
constexpr uint32_t kQueueRun = 8;
__device__ __forceinline__ uint32_t queue_slot(uint32_t b, uint32_t nb) {
    constexpr uint32_t kGroup = 8u * kQueueRun;
    const uint32_t in = b % kGroup;
    return b - in + kGroup <= nb ? b - in + (in & 7u) * kQueueRun + (in >> 3) : b;
}

// Emit position of the entry (particle with footprint u, v, r; tile tx, ty): the
// particle's offset plus the number of its member tiles before (tx, ty) in row-major
// order, counted with the same FP32 test the binning used.
__device__ __forceinline__ uint32_t emit_slot(uint32_t offset, float u, float v, float r, int tx, int ty,
                                              int tiles_x, int tiles_y, float w_lim, float h_lim) {
    int tx0, tx1, ty0, ty1;
    tile_box(u, v, r, tiles_x, tiles_y, tx0, tx1, ty0, ty1);
    const float r2 = r * r;
    uint32_t j = 0;
    for (int yy = ty0; yy <= ty; ++yy) {
        const int xe = (yy == ty) ? tx - 1 : tx1;
        for (int xx = tx0; xx <= xe; ++xx) j += tile_member(u, v, r2, xx, yy, w_lim, h_lim) ? 1u : 0u;
    }
    return offset + j;
}

// ---- Staging with 4x4 sub-blocks -----------------------------------------------------------
// Each wave owns an 8x8 quadrant; its four 16-lane rows own the quadrant's four 4x4
// sub-blocks (lane l: row g = l / 16 covers sub-block g, pixel (l % 4, (l / 4) % 4)). Every
// sub-block gets its own ordered list of the staged entries whose binning disk touches
// it, and the rows of a wave walk their lists side by side: a footprint much smaller than
// a quadrant costs a quarter of a wave step instead of a full one.
__device__ __forceinline__ int sub_x(uint32_t t) {
    return (int)(((t >> 6) & 1u) * 8u + (((t >> 4) & 3u) & 1u) * 4u + (t & 3u));
}
__device__ __forceinline__ int sub_y(uint32_t t) {
    return (int)(((t >> 6) >> 1) * 8u + (((t >> 4) & 3u) >> 1) * 4u + ((t >> 2) & 3u));
}

constexpr uint32_t kSlotBytes = 16;   // one staged float4

// The walks serve two kernel families, chosen by the template flag AN: the isotropic
// kernel of eq. 8 (a circle, one scalar 1/s^2 per entry) and the anisotropic kernel of
// eq. 5 (an ellipse: the conic A, B, C of the screen covariance of eq. 7). Staged per entry:
//   isotropic    fp {u, v, q = log2(e)/s^2, log2(o)}
//   anisotropic  fp {u, v, nA = -A log2(e), log2(o)}, cn {nB2 = -2 B log2(e), nC = -C log2(e)}
// and col {r, g, b, 0}. Both families share the footprint record's layout for
// what binning reads (centre, radius), so they share the bin sort.
template <bool AN>
struct StagedSubT {
    float4 fp[kBatch + 1];
    float4 col[kBatch + 1];
    float2 cn[AN ? kBatch + 1 : 1];
    __align__(16) uint16_t list[16][kBatch + 4];   // byte offsets (16 x staged slot) into fp and col
    __align__(16) uint32_t cnt[4][16];   // [loader wave][sub-block]
    __align__(16) uint32_t alive[4];     // [wave]: not 0 if a pixel of it is still open
};
using StagedSub = StagedSubT<false>;

// A wave's view of the staged lists: its list steps (the longest of its four rows' padded
// lists) and the padded length of this lane's row.
struct SubLists {
    uint32_t steps, len;
};

// Which sub-blocks an entry's binning disk (centre u, v, radius r) reaches: sub-block
// k = 4 * quadrant + row, quadrant q at (8 (q % 2), 8 (q / 2)) of the tile and row g of it at
// (4 (g % 2), 4 (g / 2)), holds a pixel centre within r of the centre, where the squared
// distance is a column part plus a row part; a sub-block starting beyond the image has no
// pixels. The forward and backward passes form the same FP32 sum, so they cull the same
// entries. run_distances gives the parts: squared distances of the centre coordinate c to N
// consecutive runs of four pixel centres from pixel coordinate `first` on, clipped at `lim`;
// with EDGE, a run beyond `lim` is infinitely far. Neighbouring sub-blocks share them: a tile
// takes 8 parts and 16 sums where 16 separate tests took 32 parts.
template <bool EDGE, int N>
__device__ __forceinline__ void run_distances(float c, int first, float lim, float (&d2)[N]) {
    const float base = (float)first + 0.5f;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const float lo = base + (float)(4 * q), hi = fminf(lo + 3.0f, lim);
        const float from = EDGE && lo > lim ? __builtin_inff() : lo;
        const float d = fmaxf(fmaxf(from - c, c - hi), 0.0f);
        d2[q] = d * d;
    }
}

// Whether the bit of this lane is set in the wave-uniform m: m becomes the lane mask as it is.
__device__ __forceinline__ bool lane_bit(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// `first` plus the number of set bits of m in lanes below this one.
__device__ __forceinline__ uint32_t rank_from(uint64_t m, uint32_t first) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, first));
}
// The word of a list at byte `first` (wave-uniform) plus the lane's rank in m: one shift-add.
__device__ __forceinline__ uint16_t& list_word(uint16_t* list, uint32_t first, uint64_t m) {
    return *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(list) + (first + 2u * rank_from(m, 0u)));
}

// One staged entry as loaded from global memory by its thread (k: the conic's B, C).
struct EntryLoad {
    bool ok;
    float4 f, c;
    float2 k;
};

// Staged form of an entry's kernel parameters (see StagedSubT).
template <bool AN>
__device__ __forceinline__ float4 staged_kernel(const float4& f) {
    return make_float4(f.x, f.y, (AN ? -f.z : f.z) * kLog2e, __builtin_amdgcn_logf(f.w));
}
__device__ __forceinline__ float2 staged_conic(const float2& k) {
    return make_float2(-2.0f * k.x * kLog2e, -k.y * kLog2e);
}

// alpha of a staged entry at pixel offset (dx, dy): the isotropic kernel (entry_alpha) or
// the anisotropic one, min(0.99, o exp(-(A dx^2 + 2 B dx dy + C dy^2))) evaluated as
// exp2(log2(o) + dx (nA dx + nB2 dy) + nC dy^2). `g` returns the value before the clamp.
template <bool AN>
__device__ __forceinline__ float staged_alpha(float dx, float dy, const float4& f, const float2& k, float& g) {
    if (!AN) return entry_alpha(dx, dy, f.z, f.w, g);
    const float t = fmaf(k.x, dy, f.z * dx);
    const float s = fmaf(k.y * dy, dy, f.w);
    g = __builtin_amdgcn_exp2f(fmaf(dx, t, s));
    return fminf(kAlphaMax, g);
}

// Particle index of this thread's entry of the batch at `first` (n_in_batch entries), or
// none past the end.
__device__ __forceinline__ uint32_t batch_pidx(const uint32_t* __restrict__ pidx, uint32_t first,
                                               uint32_t n_in_batch) {
    return threadIdx.x < n_in_batch ? pidx[first + threadIdx.x] : 0xFFFFFFFFu;
}

template <bool AN = false>
__device__ __forceinline__ EntryLoad load_entry(const float4* __restrict__ record, uint32_t g,
                                                uint32_t n_particles, const float2* __restrict__ conic = nullptr) {
    EntryLoad e{false, make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f), make_float2(0.f, 0.f)};
    if (g < n_particles) {
        e.ok = true;
        e.f = record[2 * (size_t)g];
        e.c = record[2 * (size_t)g + 1];
        if (AN) e.k = conic[g];
    }
    return e;
}

// Whether a pixel of the workgroup is still open, between two batches (one barrier, where
// __syncthreads_and takes two and the block's dimensions). Every wave passes `open`.
__device__ __forceinline__ bool any_alive(uint32_t (&alive)[4], bool open) {
    const uint32_t w = threadIdx.x >> 6;
    const uint64_t m = ballot64(open);
    if (lane_id() == 0) alive[w] = m != 0;
    __syncthreads();   // (the last batch's lists have been read as well)
    const uint4 v = *reinterpret_cast<const uint4*>(alive);
    return __builtin_amdgcn_readfirstlane((int)(v.x | v.y | v.z | v.w)) != 0;
}

// Stages the loaded entries of a batch (one per thread) and builds the 16 sub-block lists. The
// list positions come from scalars (the wave's ballots and the waves' counts), about four
// vector instructions per list; a wave without entries passes by. Contains __syncthreads.
template <bool AN>
__device__ __forceinline__ SubLists stage_loaded(StagedSubT<AN>& sb, const EntryLoad& e, int tile_x0, int tile_y0,
                                                 float w_lim, float h_lim) {
    const uint32_t t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = lane_id();
    const bool mine = ballot64(e.ok) != 0;
    uint64_t bal[16] = {};   // lanes whose entry joins list k
    if (mine) {
        if (e.ok) {
            sb.fp[t] = staged_kernel<AN>(e.f);
            if (AN) sb.cn[t] = staged_conic(e.k);
            sb.col[t] = make_float4(e.c.x, e.c.y, e.c.z, 0.0f);
        }
        float dxx[4], dyy[4];
        run_distances<true>(e.f.x, tile_x0, w_lim, dxx);
        run_distances<true>(e.f.y, tile_y0, h_lim, dyy);
        const float r2 = e.ok ? e.c.w * e.c.w : __builtin_nanf("");   // no entry: no comparison holds
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int qx = ((k >> 2) & 1) * 2 + (k & 1), qy = ((k >> 2) >> 1) * 2 + ((k & 3) >> 1);
            bal[k] = ballot64(dxx[qx] + dyy[qy] <= r2);
        }
    }
    if (t == 0) {
        sb.fp[kDummy] = make_float4(0.0f, 0.0f, 0.0f, -__builtin_inff());
        if (AN) sb.cn[AN ? kDummy : 0] = make_float2(0.0f, 0.0f);
        sb.col[kDummy] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    if (l == 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) sb.cnt[w][k] = (uint32_t)__popcll(bal[k]);
    }
    __syncthreads();
    // lane k (mod 16): list k's length, and the entries of earlier waves in it
    const uint32_t c0 = sb.cnt[0][l & 15u], c1 = sb.cnt[1][l & 15u], c2 = sb.cnt[2][l & 15u], c3 = sb.cnt[3][l & 15u];
    const uint32_t n = c0 + c1 + c2 + c3, padded = (n + 3u) & ~3u;
    const uint32_t before = w == 0 ? 0u : w == 1 ? c0 : w == 2 ? c0 + c1 : c0 + c1 + c2;
    if (mine) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t first = __builtin_amdgcn_readlane(2u * before, k);
            if (lane_bit(bal[k])) list_word(sb.list[k], first, bal[k]) = (uint16_t)(t * kSlotBytes);
        }
    }
    if (w == 0) {
        // pad list l / 4 with dummies up to a multiple of four, and four more: reads past the end
        const int k = (int)(l >> 2);
        const uint32_t nk = __shfl(n, k, kWave), pk = (nk + 3u) & ~3u, j = l & 3u;
        if (nk + j < pk) sb.list[k][nk + j] = (uint16_t)(kDummy * kSlotBytes);
        sb.list[k][pk + j] = (uint16_t)(kDummy * kSlotBytes);
    }
    SubLists L;
    L.len = __shfl(padded, (int)(4u * w + (l >> 4)), kWave);
    L.steps = max(max(__builtin_amdgcn_readlane(L.len, 0), __builtin_amdgcn_readlane(L.len, 16)),
                  max(__builtin_amdgcn_readlane(L.len, 32), __builtin_amdgcn_readlane(L.len, 48)));
    __syncthreads();
    return L;
}

// Loads and stages entries [first, first + n_in_batch). Contains __syncthreads.
template <bool AN>
__device__ __forceinline__ SubLists stage_batch_sub(StagedSubT<AN>& sb, const float4* __restrict__ record,
                                                    const float2* __restrict__ conic,
                                                    const uint32_t* __restrict__ pidx, uint32_t n_particles,
                                                    uint32_t first, uint32_t n_in_batch, int tile_x0, int tile_y0,
                                                    float w_lim, float h_lim) {
    return stage_loaded(sb, load_entry<AN>(record, batch_pidx(pidx, first, n_in_batch), n_particles, conic),
                        tile_x0, tile_y0, w_lim, h_lim);
}

// Byte offsets of four consecutive entries of this lane's sub-block list (padded length
// `len`) from step k; a step at or past the end reads the four dummies that follow the list.
template <bool AN>
__device__ __forceinline__ uint2 list4_sub(const StagedSubT<AN>& sb, uint32_t sbk, uint32_t k, uint32_t len) {
    return *reinterpret_cast<const uint2*>(&sb.list[sbk][min(k, len)]);
}

// Staged record of the entry at byte offset `off` (16 bytes per slot).
template <bool AN>
__device__ __forceinline__ float4 staged_fp(const StagedSubT<AN>& sb, uint32_t off) {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(sb.fp) + off);
}
// Colour component (lane % 4) of the entry at byte offset `off`.
template <bool AN>
__device__ __forceinline__ float staged_component(const StagedSubT<AN>& sb, uint32_t off) {
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(sb.col) + (off + 4u * (threadIdx.x & 3u)));
}
template <bool AN>
__device__ __forceinline__ float2 staged_cn(const StagedSubT<AN>& sb, uint32_t off) {
    if (!AN) return make_float2(0.0f, 0.0f);
    return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(sb.cn) + (off >> 1));
}

struct RenderPack {
    int32_t nv;
    uint32_t n_particles;                  // packed particles of the whole batch
    uint32_t n_entries_cap;                // entry capacity of the bins
    uint32_t block_begin[kMaxViews + 1];   // tiles of earlier views in this launch
    ViewDesc v[kMaxViews];
};

__device__ __forceinline__ void locate_tile(const RenderPack& pk, uint32_t logical, int& vi, int& tx, int& ty) {
    int v = 0;
    for (int i = 1; i < pk.nv; ++i) v = (logical >= pk.block_begin[i]) ? i : v;
    vi = __builtin_amdgcn_readfirstlane(v);
    const uint32_t local = logical - pk.block_begin[vi];
    tx = (int)(local % (uint32_t)pk.v[vi].tiles_x);
    ty = (int)(local / (uint32_t)pk.v[vi].tiles_x);
}

static inline void fill_render_pack(RenderPack& pk, const isogs_camera* cams, const int32_t* n_per_view, int v0, int nv,
                             uint32_t& p_off, uint32_t& tile_base, uint32_t& pix_off, uint32_t& blocks) {
    pk.nv = min(kMaxViews, nv - v0);
    blocks = 0;
    for (int j = 0; j < pk.nv; ++j) {
        const isogs_camera& cam = cams[v0 + j];
        ViewDesc& d = pk.v[j];
        d.p_off = p_off;
        d.n = (uint32_t)n_per_view[v0 + j];
        d.tile_base = tile_base;
        d.pix_off = pix_off;
        d.width = cam.width;
        d.height = cam.height;
        d.tiles_x = (cam.width + kTile - 1) / kTile;
        d.tiles_y = (cam.height + kTile - 1) / kTile;
        pk.block_begin[j] = blocks;
        blocks += (uint32_t)(d.tiles_x * d.tiles_y);
        p_off += d.n;
        tile_base += (uint32_t)(d.tiles_x * d.tiles_y);
        pix_off += (uint32_t)(cam.width * cam.height);
    }
    pk.block_begin[pk.nv] = blocks;
}

// Sets the batch-wide fields of a render pack.
static inline void set_render_limits(RenderPack& pk, const int32_t* n_per_view, int nv, uint64_t capacity) {
    uint64_t n = 0;
    for (int v = 0; v < nv; ++v) n += (uint64_t)n_per_view[v];
    pk.n_particles = (uint32_t)n;
    pk.n_entries_cap = (uint32_t)(capacity < 0xFFFFFFFFull ? capacity : 0xFFFFFFFFull);
}

}  // namespace isogs
