// Backward pass: gradients of a loss through compositing (eq. 4), the isotropic kernel
// (eq. 8), the projection and the spherical-harmonic colour.
//
//   1. composite_bwd  per tile: walk each pixel's entries in reverse from n_last,
//                     recovering T before each entry as T_after / (1 - alpha); reduce each
//                     entry's screen-space gradient over the tile's pixels (butterflies over
//                     the 16 pixels of a sub-block, then the sub-blocks in fixed
//                     order) into one record per entry, stored at the entry's emit position.
//   2. grad_project   per particle: sum its records (consecutive in emit order, views in
//                     order) and chain them to mu, sigma, o and the colour coefficients.
// There are no floating-point atomics: every sum has a fixed order.
#include <algorithm>
#include <array>

#include "raster.h"

namespace isogs {

// Entries staged per round, one per thread: a checkpoint chunk is one round.
constexpr int kBwdBatch = 256;
constexpr int kBwdDummy = kBwdBatch;   // staged slot of the zero-opacity pad record

// Per-entry gradient sums over a tile's pixels (dx = x - u, dy = y - v; k = dL/dalpha
// times the kernel value below the clamp, i.e. -dL/d(exponent); w = alpha T):
//   isotropic (7):    2 k dx / s^2, 2 k dy / s^2, -k d^2, k / o, dr w, dg w, db w
//   anisotropic (9):  k dx, k dy, k dx^2, k dx dy, k dy^2, k / o, dr w, dg w, db w
// (the anisotropic centre and conic gradients are these sums times the entry's conic,
// applied per particle). A record holds them in kRecVec4<AN> float4s at the entry's emit
// position.
//
// A pixel's products are formed with its own offsets and summed over the 16 pixels of a
// sub-block by a transposing butterfly, then over the sub-blocks in order. (The sums over a
// sub-block as a contraction on the matrix cores, of k with the monomials of its pixels, and
// the moments then moved to the entry's centre, take eight matrix instructions for the
// butterflies of a step, 176 us at 1080p; but the moments of a kernel narrower than a
// pixel cancel when they are moved: gradients of its scale were off by up to 1e-2.)
// Measured with the list layout below, one 1080p view of 1M particles: 254 -> 190 us;
// anisotropic 392 -> 316 us; 6M particles, eight 4K views, where most entries lie behind the
// last one composited: 8.1 -> 4.41 ms.
template <bool AN>
constexpr int kGradTerms = AN ? 9 : 7;
template <bool AN>
constexpr int kRecVec4 = AN ? 3 : 2;

// Pairs (entry, sub-block that it may touch) of a round, held in LDS list by list: the lists
// of the 16 sub-blocks lie back to back, each padded to a multiple of four, and the sums of
// the pair at list index i are part[i]. A 4x4 sub-block is touched by few of a round's
// entries (about 2 sub-blocks per entry on 1080p views of 1M particles), so a round of 256
// entries with its pairs takes less LDS than 48 entries with all 16 sub-blocks each, and the
// longer lists leave less of a wave idle: with 48 entries a wave's four lists had 2.2
// four-entry steps between two barriers. A round whose pairs exceed the capacity keeps only
// its first entries; the rest go to the next round.
// One 1080p view, four 720p views and eight 4K views of 6M particles take 190, 295 us and 4.41 ms
// with 640 pairs (31.6 KB of LDS), 201, 326 us and 4.87 ms with 672, 190 us and 4.66 ms with 896,
// 196, 320 us and 4.59 ms with 512, 211 us and 5.35 ms with 1248; anisotropic 1080p 333 us with
// 480, 320 with 528, 316 with 576 (four workgroups on a CU).
template <bool AN>
constexpr uint32_t kPairCap = AN ? 576 : 640;
constexpr uint32_t kPairPad = 16 * 3;   // padding of the 16 lists at most
template <bool AN>
constexpr int kPartPitch = AN ? 12 : 8;

template <bool AN>
struct StagedBwdT {
    float4 fp[kBwdBatch + 1];            // staged kernel (staged_kernel: {u, v, q or nA, log2(o)})
    float4 col[kBwdBatch + 1];           // {r, g, b, 1/o}
    float2 cn[AN ? kBwdBatch + 1 : 1];   // anisotropic: {nB2, nC}
    __align__(16) float part[kPairCap<AN>][kPartPitch<AN>];   // gradient sums of each pair
    __align__(16) uint32_t cnt[4][16];   // [wave][sub-block]: the wave's entries of each list
    __align__(8) uint16_t list[kPairCap<AN>];   // byte offsets (16 x staged slot) in walk order
    uint16_t link[kPairCap<AN>];         // the entry's next pair (kLinkEnd: none)
    __align__(16) uint32_t gmax[16];     // largest n_last of each sub-block
    uint32_t kept[4];
};

// An entry's pairs are chained through `link` in the order of their sub-blocks.
constexpr uint32_t kLinkEnd = 0xFFFFu;
static_assert((kBwdBatch + 1) * kSlotBytes <= 0xFFFFu, "staged byte offsets fit 16 bits");

// An entry of a round as its thread holds it.
struct BwdEntry {
    EntryLoad e;
    uint32_t slot;   // emit position (all ones: none)
    uint32_t head;   // its first pair (list index)
};

// A wave's view of the staged lists.
struct BwdLists {
    uint32_t kept;    // entries of this round
    uint32_t steps;   // list steps of the wave (the longest of its four padded lists)
    uint32_t base;    // this lane's sub-block: first list index
    uint32_t len;     // and padded length
};

// Loads the entry of this thread: staged slot t holds list position hi - 1 - t (back to front).
template <bool AN>
__device__ __forceinline__ BwdEntry load_bwd(const float4* __restrict__ record, const float2* __restrict__ conic,
                                             const uint32_t* __restrict__ pidx, const uint32_t* __restrict__ offsets,
                                             uint32_t n_particles, uint32_t hi, uint32_t nb) {
    BwdEntry b;
    const uint32_t t = threadIdx.x;
    const uint32_t g = t < nb ? pidx[hi - 1 - t] : 0xFFFFFFFFu;
    b.e = load_entry<AN>(record, g, n_particles, conic);
    b.slot = g < n_particles ? offsets[g] : 0xFFFFFFFFu;   // the particle's first; see stage_bwd
    b.head = kLinkEnd;
    return b;
}

__device__ __forceinline__ float4 staged_at(const float4* v, uint32_t off) {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(v) + off);
}

// Inclusive scan over each 16-lane row.
__device__ __forceinline__ uint32_t row_inclusive_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
    return x;
}

// Inclusive scan over the wave's lanes.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
    x = row_inclusive_scan(x);
    const uint32_t r0 = __builtin_amdgcn_readlane(x, 15), r1 = r0 + __builtin_amdgcn_readlane(x, 31),
                   r2 = r1 + __builtin_amdgcn_readlane(x, 47), l = lane_id();
    return x + (l < 16u ? 0u : l < 32u ? r0 : l < 48u ? r1 : r2);
}

// The largest value of each 16-lane row, in the row's lanes.
__device__ __forceinline__ uint32_t row_max(uint32_t x) {
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xF, 0xF, true));   // row_ror:1
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xF, 0xF, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xF, 0xF, true));
    return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true));
}

// The lanes from `first` on (64: none), in scalar registers.
__device__ __forceinline__ uint64_t lanes_from(uint32_t first) { return first < 64u ? ~0ull << first : 0ull; }

// Stages a round's entries and builds the 16 sub-block lists. An entry joins a sub-block's
// list when its binning disk reaches the sub-block (run_distances) and its position
// (pos_hi - t, 1-based) is at most the sub-block's largest n_last (no later entry was
// composited there). Contains __syncthreads.
template <bool AN>
__device__ __forceinline__ BwdLists stage_bwd(StagedBwdT<AN>& sb, BwdEntry& b, uint32_t nb, uint32_t pos_hi, int tx,
                                              int ty, int tiles_x, int tiles_y, float w_lim, float h_lim) {
    const uint32_t t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = lane_id();
    // lane k (mod 16): the wave's first lane whose entry list k takes (64: none); a sub-block
    // without pixels has gmax 0 and takes none
    const uint32_t gm = sb.gmax[l & 15u], skip = pos_hi > gm ? pos_hi - gm : 0u;
    const uint32_t from = skip > 64u * w ? min(skip - 64u * w, 64u) : 0u;
    const bool mine = ballot64(from < 64u) != 0 && 64u * w < nb;
    uint64_t bal[16] = {};   // lanes whose entry joins list k
    if (mine) {
        const float4 f = b.e.f, c = b.e.c;
        if (b.e.ok) {
            sb.fp[t] = staged_kernel<AN>(f);
            sb.col[t] = make_float4(c.x, c.y, c.z, __builtin_amdgcn_rcpf(f.w));   // once per entry
            if (AN) sb.cn[t] = staged_conic(b.e.k);
        }
        float dxx[4], dyy[4];
        run_distances<false>(f.x, tx * kTile, w_lim, dxx);
        run_distances<false>(f.y, ty * kTile, h_lim, dyy);
        const float r2 = b.e.ok ? c.w * c.w : __builtin_nanf("");   // no entry: no comparison holds
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int qx = ((k >> 2) & 1) * 2 + (k & 1), qy = ((k >> 2) >> 1) * 2 + ((k & 3) >> 1);
            bal[k] = ballot64(dxx[qx] + dyy[qy] <= r2) & lanes_from(__builtin_amdgcn_readlane(from, k));
        }
    }
    if (t == 0) {
        sb.fp[kBwdDummy] = make_float4(0.0f, 0.0f, 0.0f, -__builtin_inff());
        sb.col[kBwdDummy] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (AN) sb.cn[AN ? kBwdDummy : 0] = make_float2(0.0f, 0.0f);
    }
    BwdLists L;
    L.kept = nb;
    uint32_t n = 0, before = 0, total = 0;   // lane k (mod 16): list k's length, entries of earlier waves
    for (int attempt = 0;; ++attempt) {
        if (l == 0) {
#pragma unroll
            for (int k = 0; k < 16; ++k) sb.cnt[w][k] = (uint32_t)__popcll(bal[k]);
        }
        __syncthreads();
        const uint32_t c0 = sb.cnt[0][l & 15u], c1 = sb.cnt[1][l & 15u], c2 = sb.cnt[2][l & 15u],
                       c3 = sb.cnt[3][l & 15u];
        n = c0 + c1 + c2 + c3;
        before = (w > 0 ? c0 : 0u) + (w > 1 ? c1 : 0u) + (w > 2 ? c2 : 0u);
        total = __builtin_amdgcn_readlane(row_inclusive_scan((n + 3u) & ~3u), 15);   // with the padding
        if (attempt || total <= kPairCap<AN>) break;
        // too many pairs: keep the first entries that fit (at least (cap - pad) / 16)
        uint32_t incl = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) incl += lane_bit(bal[k]) ? 1u : 0u;
        incl = wave_inclusive_scan(incl);
        if (l == 63) sb.kept[w] = incl;
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < 3; ++q) incl += q < w ? sb.kept[q] : 0u;
        const uint64_t keep = ballot64(t < nb && incl + kPairPad <= kPairCap<AN>);
        __syncthreads();   // the wave totals have been read
        if (l == 0) sb.kept[w] = (uint32_t)__popcll(keep);
        __syncthreads();
        L.kept = sb.kept[0] + sb.kept[1] + sb.kept[2] + sb.kept[3];
#pragma unroll
        for (int k = 0; k < 16; ++k) bal[k] &= keep;
    }
    // lists back to back: lane k (mod 16) holds list k's padded length and first index
    const uint32_t padded = (n + 3u) & ~3u;
    const uint32_t base = row_inclusive_scan(padded) - padded, at = base + before;
    if (mine) {
#pragma unroll
        for (int k = 15; k >= 0; --k) {
            const uint32_t first = __builtin_amdgcn_readlane(at, k);
            if (lane_bit(bal[k])) {
                const uint32_t i = first + rank_from(bal[k], 0u);
                sb.list[i] = (uint16_t)(t * kSlotBytes);
                sb.link[i] = (uint16_t)b.head;
                b.head = i;
            }
        }
        if (b.head != kLinkEnd)
            b.slot = emit_slot(b.slot, b.e.f.x, b.e.f.y, b.e.c.w, tx, ty, tiles_x, tiles_y, w_lim, h_lim);
    }
    if (w == 0) {
        // pad list l / 4 with dummies
        const int k = (int)(l >> 2);
        const uint32_t i = __shfl(n, k, 64) + (l & 3u), pk = __shfl(padded, k, 64), bk = __shfl(base, k, 64);
        if (i < pk) sb.list[bk + i] = (uint16_t)(kBwdDummy * kSlotBytes);
    }
    const int sbk = (int)(4u * w + (l >> 4));
    L.base = __shfl(base, sbk, 64);
    L.len = __shfl(padded, sbk, 64);
    const uint32_t most = max(max(__builtin_amdgcn_readlane(L.len, 0), __builtin_amdgcn_readlane(L.len, 16)),
                              max(__builtin_amdgcn_readlane(L.len, 32), __builtin_amdgcn_readlane(L.len, 48)));
    L.steps = total ? most : 0u;
    __syncthreads();
    return L;
}

// Reverse walk of one tile (logical index within the launch) by a 256-thread workgroup,
// one lane per pixel, each 16-lane row owning a 4x4 sub-block (the forward pixel layout).
// Record of an entry: its gradient sums (kGradTerms), at its emit position, marked in
// has_rec; an entry that no pixel composited has neither.
// With checkpoints (`ckpt` non-null) and a list of at least kChunkedMin entries, the
// workgroup walks only chunk `chunk` of the list, positions [chunk * kCkptChunk,
// (chunk + 1) * kCkptChunk); a pixel whose last entry lies beyond the chunk starts from the
// checkpoint at the chunk's end: T from there, and the light from behind = image - colour
// accumulated before the chunk's end. Shorter lists, and every list without checkpoints,
// are one chunk. Contains __syncthreads.
template <bool AN>
__device__ __forceinline__ void composite_bwd_tile(
    StagedBwdT<AN>& sb, const RenderPack& pk, uint32_t logical, uint32_t chunk, const float4* __restrict__ record,
    const float2* __restrict__ conic, const uint32_t* __restrict__ pidx, const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ ranges,
    float bg_r, float bg_g, float bg_b, const float* __restrict__ image, const float* __restrict__ dL_dimage,
    const float* __restrict__ T_final, const uint32_t* __restrict__ n_last, const float4* __restrict__ ckpt,
    float4* __restrict__ rec, uint8_t* __restrict__ has_rec) {
    int vi, tx, ty;
    locate_tile(pk, logical, vi, tx, ty);
    const ViewDesc& vd = pk.v[vi];
    const uint32_t t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), lane = lane_id();
    const uint32_t sbk = 4 * w + ((t >> 4) & 3u);   // this lane's sub-block
    const int x = tx * kTile + sub_x(t), y = ty * kTile + sub_y(t);
    const bool inside = x < vd.width && y < vd.height;
    const float px = (float)x + 0.5f, py = (float)y + 0.5f;
    const uint32_t gt = vd.tile_base + (uint32_t)(ty * vd.tiles_x + tx);
    const uint32_t start = ranges[2 * gt], end = min(ranges[2 * gt + 1], pk.n_entries_cap);
    const float w_lim = (float)vd.width - 0.5f, h_lim = (float)vd.height - 0.5f;
    const uint32_t len = end > start ? end - start : 0u;
    // this workgroup's positions [c_lo, c_hi) of the list
    const bool chunked = ckpt && chunked_list(len);
    const uint32_t c_lo = chunked ? chunk * kCkptChunk : 0u;
    const uint32_t c_hi = chunked ? min(c_lo + kCkptChunk, len) : len;
    if (c_lo >= c_hi) return;   // no such chunk, or an empty list (uniform over the workgroup)

    // the first round's entries are loaded beside the pixels
    uint32_t hi = start + c_hi, nb = min((uint32_t)kBwdBatch, c_hi - c_lo);
    BwdEntry b = load_bwd<AN>(record, conic, pidx, offsets, pk.n_particles, hi, nb);

    // S: light from behind the current entry, per channel
    float T = 1.0f, dr = 0.0f, dg = 0.0f, db = 0.0f, Sr = 0.0f, Sg = 0.0f, Sb = 0.0f;
    uint32_t last = 0;
    if (inside) {
        const size_t hw = (size_t)vd.width * vd.height;
        const size_t pix = (size_t)y * vd.width + x;
        const float* dimg = dL_dimage + (size_t)3 * vd.pix_off;
        dr = dimg[pix];
        dg = dimg[hw + pix];
        db = dimg[2 * hw + pix];
        last = n_last[vd.pix_off + pix];
        if (last > c_hi) {
            // the pixel composited entries beyond this chunk: state at the chunk's end
            const float4 s = ckpt[(size_t)ckpt_slot(start, c_hi / kCkptChunk) * 256 + t];
            const float* im = image + (size_t)3 * vd.pix_off;
            T = s.x;
            Sr = im[pix] - s.y;
            Sg = im[hw + pix] - s.z;
            Sb = im[2 * hw + pix] - s.w;
        } else {
            // light arriving from behind the last entry: T_final bg
            T = T_final[vd.pix_off + pix];
            Sr = T * bg_r;
            Sg = T * bg_g;
            Sb = T * bg_b;
        }
    }

    const uint32_t most = row_max(last > c_lo ? min(last, c_hi) : 0u);
    if ((lane & 15u) == 0) sb.gmax[sbk] = most;
    __syncthreads();
    if (ballot64(sb.gmax[lane & 15u] != 0u) == 0) return;   // no pixel composited an entry from here on

    // this lane's sum of its row (anisotropic: the ninth in lane 8)
    const uint32_t q8 = rev3(lane & 7u);
    const bool writer8 = (lane & 15u) < 8u, writer9 = AN && (lane & 15u) == 8u;

    while (true) {
        const uint32_t pos_hi = hi - start;
        const BwdLists L = stage_bwd(sb, b, nb, pos_hi, tx, ty, vd.tiles_x, vd.tiles_y, w_lim, h_lim);
        // staged slot j holds list position pos_hi - j (1-based): composited by this pixel
        // in the forward pass only from slot pos_hi - last on
        const int off_min = ((int)pos_hi - (int)last) * (int)kSlotBytes;
        for (uint32_t k = 0; k < L.steps; k += 4) {
            constexpr uint64_t kD = (uint64_t)kBwdDummy * kSlotBytes;
            uint64_t q4 = kD | (kD << 16) | (kD << 32) | (kD << 48);   // four dummy slots
            const bool on = k < L.len;
            if (on) q4 = *reinterpret_cast<const uint64_t*>(&sb.list[L.base + k]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t off = (uint32_t)(q4 >> (16 * r)) & 0xFFFFu;
                const float4 f = staged_at(sb.fp, off), c = staged_at(sb.col, off);
                const float2 kc = AN ? sb.cn[off / kSlotBytes] : make_float2(0.0f, 0.0f);
                const float dx = px - f.x, dy = py - f.y;
                float ga;
                float a = staged_alpha<AN>(dx, dy, f, kc, ga);
                // an entry this pixel composited in the forward pass (same decision); the
                // pad record has alpha 0
                const bool use = (int)off >= off_min && a >= kAlphaMin;
                a = use ? a : 0.0f;
                const float inv_om = __builtin_amdgcn_rcpf(1.0f - a);
                T = T * inv_om;                              // transmittance before this entry
                const float wgt = a * T;
                const float dLda = dr * (c.x * T - Sr * inv_om) + dg * (c.y * T - Sg * inv_om) +
                                   db * (c.z * T - Sb * inv_om);
                Sr = fmaf(c.x, wgt, Sr);
                Sg = fmaf(c.y, wgt, Sg);
                Sb = fmaf(c.z, wgt, Sb);
                // alpha = o exp(-d^2 / s^2) below the clamp: d/du = 2 alpha dx / s^2,
                // d/d(1/s^2) = -alpha d^2, d/do = alpha / o
                const float kk = (use && ga < kAlphaMax) ? dLda * ga : 0.0f;
                float red = 0.0f, g9 = 0.0f;
                if (ballot64(use) != 0) {
                    float gv[8];
                    if constexpr (!AN) {
                        const float inv_s2 = f.z * (1.0f / kLog2e);
                        gv[0] = 2.0f * kk * inv_s2 * dx;
                        gv[1] = 2.0f * kk * inv_s2 * dy;
                        gv[2] = -kk * fmaf(dx, dx, dy * dy);
                        gv[3] = kk * c.w;
                        gv[4] = dr * wgt;
                        gv[5] = dg * wgt;
                        gv[6] = db * wgt;
                        gv[7] = 0.0f;
                    } else {
                        // alpha = o exp(-Q) below the clamp: dL/du = k (2 A dx + 2 B dy),
                        // dL/dA = -k dx^2, ...: the conic enters per particle
                        const float kx = kk * dx, ky = kk * dy;
                        gv[0] = kx;
                        gv[1] = ky;
                        gv[2] = kx * dx;
                        gv[3] = kx * dy;
                        gv[4] = ky * dy;
                        gv[5] = kk * c.w;
                        gv[6] = dr * wgt;
                        gv[7] = dg * wgt;
                        // the ninth sum over the row: butterfly (quad swaps, row rotations)
                        g9 = db * wgt;
                        g9 += dpp<0xB1>(g9);
                        g9 += dpp<0x4E>(g9);
                        g9 += dpp<0x124>(g9);
                        g9 += dpp<0x128>(g9);
                    }
                    red = row_sum8(gv, lane);
                }
                // the sums of pads are written too (nothing reads them)
                float* pr = sb.part[on ? L.base + k + r : 0u];
                if (on && writer8) pr[q8] = red;
                if (on && writer9) pr[AN ? 8 : 0] = g9;
            }
        }
        __syncthreads();
        // combine: each thread sums its entry's pairs in the order of the sub-blocks
        if (b.head != kLinkEnd && b.slot < pk.n_entries_cap) {
            constexpr int kSums = kGradTerms<AN>;
            float sum[4 * kRecVec4<AN>] = {};
            for (uint32_t next = b.head; next != kLinkEnd;) {
                const float* p = sb.part[next];
                next = sb.link[next];
#pragma unroll
                for (int q = 0; q < kSums; ++q) sum[q] += p[q];
            }
            float4* r = rec + kRecVec4<AN> * (size_t)b.slot;
#pragma unroll
            for (int q = 0; q < kRecVec4<AN>; ++q)
                r[q] = make_float4(sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]);
            has_rec[b.slot] = 1;
        }
        hi -= L.kept;
        if (hi <= start + c_lo) break;
        nb = min((uint32_t)kBwdBatch, hi - start - c_lo);
        b = load_bwd<AN>(record, conic, pidx, offsets, pk.n_particles, hi, nb);
        __syncthreads();   // the staged round has been read
    }
}

__global__ void __launch_bounds__(64) fill_u32_kernel_b(uint32_t* __restrict__ p, uint32_t n) {
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

__global__ void __launch_bounds__(256) clear_marks_kernel(uint8_t* __restrict__ marks,
                                                          const uint32_t* __restrict__ count_p, uint64_t capacity) {
    // (the marks are 256-byte aligned and padded to whole 16-byte vectors)
    const uint64_t n = min((uint64_t)*count_p, capacity);
    for (uint64_t i = ((uint64_t)blockIdx.x * 256u + threadIdx.x) * 16u; i < n; i += (uint64_t)gridDim.x * 4096u)
        *reinterpret_cast<uint4*>(marks + i) = make_uint4(0u, 0u, 0u, 0u);
}

// Work items of the tiles whose list is longer than one checkpoint chunk: one (tile, chunk)
// pair per chunk up to the last that a pixel of the tile composited from (occluded entries,
// most of the long lists of dense scenes, then cost no workgroup), appended in any order,
// with one device-wide add per workgroup (adds to one counter from many XCDs are serialised
// in memory). A workgroup takes 64 tiles; 16 lanes read a tile's n_last, a row each.
constexpr uint32_t kReachTiles = 64;

__global__ void __launch_bounds__(256) bwd_chunk_list_kernel(const RenderPack pk, const uint32_t* __restrict__ ranges,
                                                             uint32_t tile0, uint32_t n_tiles,
                                                             const uint32_t* __restrict__ n_last,
                                                             const int32_t* __restrict__ status,
                                                             uint32_t* __restrict__ heavy,
                                                             uint32_t* __restrict__ heavy_count,
                                                             uint32_t heavy_max) {
    __shared__ uint32_t s_n[kReachTiles];
    if (*status != kStatusOk) return;
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6, r = lane & 15u;
#pragma unroll
    for (uint32_t q = 0; q < kReachTiles / 16; ++q) {
        const uint32_t at = 16u * q + 4u * w + (lane >> 4);   // tile of this row of lanes
        const uint32_t i = blockIdx.x * kReachTiles + at;
        uint32_t most = 0, len = 0;
        if (i < n_tiles) {
            const uint32_t s = ranges[2 * (tile0 + i)], e = min(ranges[2 * (tile0 + i) + 1], pk.n_entries_cap);
            len = e > s ? e - s : 0u;
        }
        if (chunked_list(len)) {
            int v = 0;
            for (int j = 1; j < pk.nv; ++j) v = i >= pk.block_begin[j] ? j : v;
            const ViewDesc& vd = pk.v[v];
            const uint32_t local = i - pk.block_begin[v];
            const int x0 = (int)(local % (uint32_t)vd.tiles_x) * kTile;
            const int y = (int)(local / (uint32_t)vd.tiles_x) * kTile + (int)r;
            if (y < vd.height) {
                const uint32_t* p = n_last + vd.pix_off + (size_t)y * vd.width + x0;
                if (x0 + kTile <= vd.width && (reinterpret_cast<uintptr_t>(p) & 15u) == 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint4 n = reinterpret_cast<const uint4*>(p)[c];
                        most = max(most, max(max(n.x, n.y), max(n.z, n.w)));
                    }
                } else {
                    for (int c = 0; c < min(kTile, vd.width - x0); ++c) most = max(most, p[c]);
                }
            }
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o, 16));
        if (r == 0) s_n[at] = chunked_list(len) ? (min(most, len) + kCkptChunk - 1) / kCkptChunk : 0u;
    }
    __syncthreads();
    if (w != 0) return;
    const uint32_t nch = s_n[lane];
    uint32_t incl = nch;
#pragma unroll
    for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    const uint32_t total = __shfl(incl, 63, 64);
    uint32_t base = 0;
    if (lane == 0 && total) base = atomicAdd(heavy_count, total);
    base = __shfl(base, 0, 64) + incl - nch;
    if (!nch || base + nch > heavy_max) return;   // the bound holds for ranges that partition the entries
    const uint32_t i = blockIdx.x * kReachTiles + lane;
    for (uint32_t c = 0; c < nch; ++c) {
        heavy[2 * (base + c)] = i;
        heavy[2 * (base + c) + 1] = c;
    }
}

// One workgroup per work item, in dispatch order. With checkpoints: workgroups
// [0, n_chunks) take the reached chunks of the long tiles (listed by bwd_chunk_list_kernel), the
// next ones the other tiles in longest-list-first order (they follow the long ones in the
// queue, whose length classes tell how many those are); a workgroup past the last item
// leaves at once. Without: workgroup b walks the tile at queue position b whole.
struct BwdArgs {
    const float4* record;
    const float2* conic;     // anisotropic family: {B, C} per record
    const uint32_t* pidx;
    const uint32_t* offsets;
    const uint32_t* ranges;
    const int32_t* status;
    float bg_r, bg_g, bg_b;
    const float* image;
    const float* dL_dimage;
    const float* T_final;
    const uint32_t* n_last;
    const float4* ckpt;
    float4* rec;
    uint8_t* has_rec;
    const uint32_t* order;
    const uint32_t* hist;
    uint32_t n_items;
    const uint32_t* heavy;
    const uint32_t* heavy_count;
    uint32_t heavy_max;
};

// LOOP: a workgroup takes every gridDim.x-th item. Otherwise it takes one, and leaves at once
// past the last: the number of items is known on the device only, at most tiles + capacity /
// kCkptChunk, and where much of the lists lies behind opaque particles most workgroups find none,
// after waiting for LDS and two loads (two thirds of 760 thousand in eight 4K views of 6M
// particles, with 16384 to 131072 workgroups alike; the 1024 that reside are 6% slower). The
// loop costs registers and a barrier per item, so it is for launches of more than kBwdLoopItems.
// Without and with it: 1080p views of 1M particles, one (17 thousand items) 245 and 246 us, four (67)
// 761 and 776, ten (166) 1.87 and 1.92 ms, 16 (265) 3.06 and 3.11, 20 (298) 3.90 and 3.91; eight 4K
// views (370) 3.45 and 3.43, of 6M particles four (382) 2.54 and 2.52, eight (766) 5.14 and 5.04.
constexpr uint32_t kBwdLoopGrid = 32768, kBwdLoopItems = 10 * kBwdLoopGrid;

template <bool AN, bool LOOP>
__device__ __forceinline__ void bwd_ordered(StagedBwdT<AN>& sb, const RenderPack& pk, const BwdArgs& A) {
    if (*A.status != kStatusOk) return;
    const uint32_t n_heavy = A.ckpt ? min(*A.heavy_count, A.heavy_max) : 0u;
    uint32_t b = blockIdx.x;
    do {
        uint32_t logical, chunk = 0;
        if (b < n_heavy) {
            logical = A.heavy[2 * b];
            chunk = A.heavy[2 * b + 1];
            if (logical >= A.n_items) return;
        } else {
            uint32_t n_long = 0;
            if (A.ckpt)
                for (int c = kChunkedClass; c < kBuckets; ++c) n_long += A.hist[c];
            const uint32_t j = n_long + (b - n_heavy);
            if (j >= A.n_items) return;
            logical = A.order[j];
        }
        composite_bwd_tile(sb, pk, logical, chunk, A.record, A.conic, A.pidx, A.offsets, A.ranges, A.bg_r, A.bg_g,
                           A.bg_b, A.image, A.dL_dimage, A.T_final, A.n_last, A.ckpt, A.rec, A.has_rec);
        if (LOOP) __syncthreads();   // the item's LDS has been read
        b += gridDim.x;
    } while (LOOP);
}

template <bool LOOP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
composite_bwd_ordered_kernel(const RenderPack pk, const BwdArgs a) {
    __shared__ StagedBwdT<false> sb;
    bwd_ordered<false, LOOP>(sb, pk, a);
}

// The anisotropic family (eq. 5 kernels).
template <bool LOOP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
aniso_bwd_ordered_kernel(const RenderPack pk, const BwdArgs a) {
    __shared__ StagedBwdT<true> sb;
    bwd_ordered<true, LOOP>(sb, pk, a);
}

struct GradView {
    uint32_t p_off;
    float R[9], t[3], eye[3], f, cx, cy;
};

// Real SH basis polynomial K (the forms of the forward colour evaluation) and its gradient
// at direction (x, y, z); K is a compile-time constant, so each call folds to its own term.
template <int K>
__device__ __forceinline__ void sh_term(float x, float y, float z, float& Y, float& gx, float& gy, float& gz) {
    constexpr float c1 = 0.48860251190291992f, c2a = 1.09254843059207907f, c2b = 0.31539156525252005f,
                    c2c = 0.54627421529603959f, c3a = 0.59004358992664352f, c3b = 2.89061144264055405f,
                    c3c = 0.45704579946446573f, c3d = 0.37317633259011540f, c3e = 1.44530572132027702f;
    const float xx = x * x, yy = y * y, zz = z * z;
    gx = gy = gz = 0.0f;
    if constexpr (K == 1) { Y = c1 * y; gy = c1; }
    else if constexpr (K == 2) { Y = c1 * z; gz = c1; }
    else if constexpr (K == 3) { Y = c1 * x; gx = c1; }
    else if constexpr (K == 4) { Y = c2a * x * y; gx = c2a * y; gy = c2a * x; }
    else if constexpr (K == 5) { Y = c2a * y * z; gy = c2a * z; gz = c2a * y; }
    else if constexpr (K == 6) { Y = c2b * (3.0f * zz - 1.0f); gz = 6.0f * c2b * z; }
    else if constexpr (K == 7) { Y = c2a * x * z; gx = c2a * z; gz = c2a * x; }
    else if constexpr (K == 8) { Y = c2c * (xx - yy); gx = 2.0f * c2c * x; gy = -2.0f * c2c * y; }
    else if constexpr (K == 9) { Y = c3a * y * (3.0f * xx - yy); gx = 6.0f * c3a * x * y; gy = 3.0f * c3a * (xx - yy); }
    else if constexpr (K == 10) { Y = c3b * x * y * z; gx = c3b * y * z; gy = c3b * x * z; gz = c3b * x * y; }
    else if constexpr (K == 11) { Y = c3c * y * (5.0f * zz - 1.0f); gy = c3c * (5.0f * zz - 1.0f); gz = 10.0f * c3c * y * z; }
    else if constexpr (K == 12) { Y = c3d * z * (5.0f * zz - 3.0f); gz = c3d * (15.0f * zz - 3.0f); }
    else if constexpr (K == 13) { Y = c3c * x * (5.0f * zz - 1.0f); gx = c3c * (5.0f * zz - 1.0f); gz = 10.0f * c3c * x * z; }
    else if constexpr (K == 14) { Y = c3e * z * (xx - yy); gx = 2.0f * c3e * x * z; gy = -2.0f * c3e * y * z; gz = c3e * (xx - yy); }
    else { static_assert(K == 15, "degree 3 at most"); Y = c3a * x * (xx - 3.0f * yy); gx = 3.0f * c3a * (xx - yy); gy = -6.0f * c3a * x * y; }
}

// The coefficients of one particle, held in registers across the views: coefficient k of
// channel ch at c[3 k + ch].
struct CoefRef {
    const float* c;
    __device__ float operator()(int k, int ch) const { return c[3 * k + ch]; }
};

// Colour of one view, rgb = max(0, c_0 + sum_k c_k Y_k(d)) with d = (mu - eye)/|mu - eye|:
// adds the view's gradient (drgb, zero where the colour was clamped) to the coefficients'
// and to the centre's (through the direction's tangential part). Each channel's sum runs
// over k in ascending order, as in the forward evaluation, so the clamp decision agrees.
template <int DEG, int KK = 1>
__device__ __forceinline__ void sh_raw(const CoefRef& coef, float x, float y, float z, float raw[3]) {
    if constexpr (KK < (DEG + 1) * (DEG + 1)) {
        float Y, gx, gy, gz;
        sh_term<KK>(x, y, z, Y, gx, gy, gz);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) raw[ch] = fmaf(coef(KK, ch), Y, raw[ch]);
        sh_raw<DEG, KK + 1>(coef, x, y, z, raw);
    }
}

// Bit k: Y_k depends on x, y, z (sh_term sets that derivative).
constexpr uint32_t kShDx = 0xE798u, kShDy = 0xCF32u, kShDz = 0x7CE4u;

template <int DEG, int KK = 1>
__device__ __forceinline__ void sh_back(const CoefRef& coef, float x, float y, float z, const float d[3], float* gcol,
                                        float& wdx, float& wdy, float& wdz) {
    if constexpr (KK < (DEG + 1) * (DEG + 1)) {
        float Y, gx, gy, gz;
        sh_term<KK>(x, y, z, Y, gx, gy, gz);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) gcol[3 * KK + ch] = fmaf(d[ch], Y, gcol[3 * KK + ch]);
        // dL/dY_k, then along its derivatives (those that are not identically zero)
        const float wk = fmaf(d[2], coef(KK, 2), fmaf(d[1], coef(KK, 1), d[0] * coef(KK, 0)));
        if constexpr ((kShDx >> KK) & 1u) wdx = fmaf(wk, gx, wdx);
        if constexpr ((kShDy >> KK) & 1u) wdy = fmaf(wk, gy, wdy);
        if constexpr ((kShDz >> KK) & 1u) wdz = fmaf(wk, gz, wdz);
        sh_back<DEG, KK + 1>(coef, x, y, z, d, gcol, wdx, wdy, wdz);
    }
}

template <int DEG>
__device__ __forceinline__ void color_backward(const CoefRef& coef, const float drgb[3], const float eye[3], float mx,
                                               float my, float mz, float* gcol, float& gmx, float& gmy, float& gmz) {
    const float ex = mx - eye[0], ey = my - eye[1], ez = mz - eye[2];
    const float inv_dist = 1.0f / sqrtf(ex * ex + ey * ey + ez * ez);
    const float dxn = ex * inv_dist, dyn = ey * inv_dist, dzn = ez * inv_dist;
    float raw[3] = {coef(0, 0), coef(0, 1), coef(0, 2)};
    sh_raw<DEG>(coef, dxn, dyn, dzn, raw);
    float d[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        d[ch] = (raw[ch] > 0.0f) ? drgb[ch] : 0.0f;
        gcol[ch] += d[ch];
    }
    float wdx = 0.0f, wdy = 0.0f, wdz = 0.0f;
    sh_back<DEG>(coef, dxn, dyn, dzn, d, gcol, wdx, wdy, wdz);
    const float radial = wdx * dxn + wdy * dyn + wdz * dzn;
    gmx += (wdx - radial * dxn) * inv_dist;
    gmy += (wdy - radial * dyn) * inv_dist;
    gmz += (wdz - radial * dzn) * inv_dist;
}

struct GradPack {
    int32_t nv;            // views of this scene in this launch, in view order
    int32_t accumulate;    // add to the outputs (a previous launch covered earlier views)
    const float* pos;
    const float* scale;
    const float* opacity;
    const float* color;
    uint32_t n;
    int32_t sh_degree;
    float* g_pos;
    float* g_scale;
    float* g_opacity;
    float* g_color;
    GradView v[kMaxViews];
};

// The records of a workgroup's 256 particles in one view are one run of the emit order
// (offsets are a scan of the tile counts). The run is staged in LDS window by window with
// coalesced loads (marked records only, zeros for the others) and each thread adds its own
// particle's records from there, in emit order. Read by each thread from global memory, the
// record loop of a wave lasted as long as its particle with the most tiles, a load latency
// per turn: 6M particles x 8 views of 4K took 2329 us (2989 us with marks read first).
constexpr uint32_t kRecWindow = 512;

template <int NV>
struct RecShared {
    float4 v[NV][kRecWindow];
    uint32_t run[2];
    __align__(16) uint32_t marked[4];   // [wave]: not 0 if it staged a marked record
};

// Sums the NV float4s of records [e0, e0 + cnt) into S (zeroed here). Every thread of the
// workgroup calls it, e0 non-decreasing over the threads; false: no record was marked.
// Contains __syncthreads.
template <int NV>
__device__ __forceinline__ bool sum_records(RecShared<NV>& sh, const float4* __restrict__ rec,
                                            const uint8_t* __restrict__ has_rec, uint32_t e0, uint32_t cnt,
                                            float (&S)[4 * NV]) {
    const uint32_t t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 4 * NV; ++k) S[k] = 0.0f;
    if (t == 0) sh.run[0] = e0;
    if (t == 255) sh.run[1] = e0 + cnt;
    __syncthreads();
    const uint32_t lo = sh.run[0], hi = sh.run[1];
    bool any = false;
    for (uint32_t w0 = lo; w0 < hi; w0 += kRecWindow) {
        bool has[kRecWindow / 256];
#pragma unroll
        for (uint32_t q = 0; q < kRecWindow / 256; ++q) {
            const uint32_t e = w0 + q * 256u + t;
            has[q] = e < hi && has_rec[e];
        }
#pragma unroll
        for (uint32_t q = 0; q < kRecWindow / 256; ++q) {
            float4 r[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) r[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (has[q]) {
#pragma unroll
                for (int k = 0; k < NV; ++k) r[k] = rec[NV * (size_t)(w0 + q * 256u + t) + k];
            }
#pragma unroll
            for (int k = 0; k < NV; ++k) sh.v[k][q * 256u + t] = r[k];
        }
        const uint64_t marked = ballot64(has[0] || has[1]);
        if (lane_id() == 0) sh.marked[t >> 6] = marked != 0;
        __syncthreads();
        const uint4 m = *reinterpret_cast<const uint4*>(sh.marked);
        if (__builtin_amdgcn_readfirstlane((int)(m.x | m.y | m.z | m.w))) {
            any = true;
            for (uint32_t e = max(e0, w0); e < min(e0 + cnt, w0 + kRecWindow); ++e) {
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const float4 r = sh.v[k][e - w0];
                    S[4 * k] += r.x;
                    S[4 * k + 1] += r.y;
                    S[4 * k + 2] += r.z;
                    S[4 * k + 3] += r.w;
                }
            }
        }
        __syncthreads();   // the window has been read (and, before the next view, the run)
    }
    static_assert(kRecWindow == 512, "two records per thread and window");
    if (lo >= hi) __syncthreads();   // uniform: the run has been read
    return any;
}

// The entries of a particle in one view, clipped to a valid run: [e0, e0 + cnt).
struct RecRun {
    uint32_t e0, cnt;
};

__device__ __forceinline__ RecRun record_run(const uint32_t* __restrict__ tile_count,
                                             const uint32_t* __restrict__ offsets, uint32_t pi, bool in,
                                             uint32_t n_entries) {
    RecRun r{offsets[pi], tile_count[pi]};
    if ((uint64_t)r.e0 + r.cnt > n_entries) r = {min(r.e0, n_entries), 0u};
    if (!in) r = {r.e0 + r.cnt, 0u};   // behind the last particle's
    return r;
}

// One thread per particle of one scene; DEG is the scene's SH degree. The records, parameters
// and gradients of one view of 1M particles (480 MB) take 89 us, the rate of a copy; eight views
// wait on each view's marks and records in turn: 6M particles 1.90 -> 1.74 ms with a quarter fewer
// vector instructions (one sum over the channels per coefficient, derivatives that are zero left
// out, one FP64 division).
template <int DEG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) grad_project_kernel(const GradPack pk, const float4* __restrict__ rec,
                                                           const uint8_t* __restrict__ has_rec,
                                                           const uint32_t* __restrict__ tile_count,
                                                           const uint32_t* __restrict__ offsets,
                                                           const uint32_t* __restrict__ count_p,
                                                           const int32_t* __restrict__ status) {
    __shared__ RecShared<kRecVec4<false>> sh;
    if (*status != kStatusOk) return;
    const uint32_t n_entries = *count_p;
    // threads past the last particle stay for the shared record sums, on the last one's inputs
    const bool in = blockIdx.x * 256u + threadIdx.x < pk.n;
    const uint32_t i = min(blockIdx.x * 256u + threadIdx.x, pk.n - 1u);
    const uint32_t n = pk.n;
    constexpr int K = (DEG + 1) * (DEG + 1);
    const float mx = pk.pos[i], my = pk.pos[n + i], mz = pk.pos[2 * n + i];
    const float sigma = pk.scale[i];

    float gmx = 0.0f, gmy = 0.0f, gmz = 0.0f, gsig = 0.0f, gop = 0.0f;
    float gcol[3 * K];
    float coef[3 * K];
#pragma unroll
    for (int k = 0; k < 3 * K; ++k) {
        gcol[k] = 0.0f;
        coef[k] = pk.color[(size_t)k * n + i];
    }

    RecRun next = record_run(tile_count, offsets, pk.v[0].p_off + i, in, n_entries);
    for (int vv = 0; vv < pk.nv; ++vv) {
        const GradView& gv = pk.v[vv];
        const RecRun cur = next;
        if (vv + 1 < pk.nv) next = record_run(tile_count, offsets, pk.v[vv + 1].p_off + i, in, n_entries);
        float S[8];
        if (!sum_records<2>(sh, rec, has_rec, cur.e0, cur.cnt, S) || cur.cnt == 0) continue;
        const float du = S[0], dv = S[1], dis2 = S[2], dop = S[3], drgb[3] = {S[4], S[5], S[6]};
        gop += dop;
        // projection: p = R mu + t, u = f p_x/z + cx, v = f p_y/z + cy, s = f sigma/z, 1/s^2
        const double pxd = (double)gv.R[0] * mx + (double)gv.R[1] * my + (double)gv.R[2] * mz + (double)gv.t[0];
        const double pyd = (double)gv.R[3] * mx + (double)gv.R[4] * my + (double)gv.R[5] * mz + (double)gv.t[1];
        const double pzd = (double)gv.R[6] * mx + (double)gv.R[7] * my + (double)gv.R[8] * mz + (double)gv.t[2];
        const double izd = 1.0 / pzd;   // (one FP64 division; the quotients below are rounded to FP32)
        const float inv_z = (float)izd;
        const float s = (float)((double)gv.f * (double)sigma * izd);
        const float inv_s = 1.0f / s;
        // d(1/s^2)/ds = -2/s^3
        const float ds = -2.0f * dis2 * inv_s * inv_s * inv_s;
        gsig += ds * gv.f * inv_z;
        const float gpx = du * gv.f * inv_z, gpy = dv * gv.f * inv_z;
        const float ucx = (float)((double)gv.f * pxd * izd), vcy = (float)((double)gv.f * pyd * izd);
        const float gpz = -(ds * s + du * ucx + dv * vcy) * inv_z;
        gmx += gv.R[0] * gpx + gv.R[3] * gpy + gv.R[6] * gpz;
        gmy += gv.R[1] * gpx + gv.R[4] * gpy + gv.R[7] * gpz;
        gmz += gv.R[2] * gpx + gv.R[5] * gpy + gv.R[8] * gpz;
        color_backward<DEG>(CoefRef{coef}, drgb, gv.eye, mx, my, mz, gcol, gmx, gmy, gmz);
    }
    if (!in) return;
    if (pk.accumulate) {
        pk.g_pos[i] += gmx;
        pk.g_pos[n + i] += gmy;
        pk.g_pos[2 * n + i] += gmz;
        pk.g_scale[i] += gsig;
        pk.g_opacity[i] += gop;
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) pk.g_color[(size_t)k * n + i] += gcol[k];
    } else {
        pk.g_pos[i] = gmx;
        pk.g_pos[n + i] = gmy;
        pk.g_pos[2 * n + i] = gmz;
        pk.g_scale[i] = gsig;
        pk.g_opacity[i] = gop;
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) pk.g_color[(size_t)k * n + i] = gcol[k];
    }
}

// ---- Anisotropic chain rule (eq. 5-7) ------------------------------------------------------
struct AnisoGradPack {
    int32_t nv;            // views of this scene in this launch, in view order
    int32_t accumulate;    // add to the outputs (a previous launch covered earlier views)
    const float* pos;
    const float* rot;
    const float* scale;
    const float* opacity;
    const float* color;
    uint32_t n;
    int32_t sh_degree;
    float* g_pos;
    float* g_rot;
    float* g_scale;
    float* g_opacity;
    float* g_color;
    GradView v[kMaxViews];
};

// Rotation matrix of the unit quaternion (w, x, y, z), row-major.
__device__ __forceinline__ void quat_rot(double w, double x, double y, double z, double R[9]) {
    R[0] = 1.0 - 2.0 * (y * y + z * z); R[1] = 2.0 * (x * y - w * z);       R[2] = 2.0 * (x * z + w * y);
    R[3] = 2.0 * (x * y + w * z);       R[4] = 1.0 - 2.0 * (x * x + z * z); R[5] = 2.0 * (y * z - w * x);
    R[6] = 2.0 * (x * z - w * y);       R[7] = 2.0 * (y * z + w * x);       R[8] = 1.0 - 2.0 * (x * x + y * y);
}

// Particle i's colour gradients (added to the outputs if an earlier launch wrote them).
template <int K>
__device__ __forceinline__ void store_color(const AnisoGradPack& pk, uint32_t i, const float (&gcol)[3 * K]) {
    const size_t n = pk.n;
    if (pk.accumulate) {
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) pk.g_color[k * n + i] += gcol[k];
    } else {
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) pk.g_color[k * n + i] = gcol[k];
    }
}

// Index of element (a, b) of a symmetric 3 x 3 matrix held as xx, xy, xz, yy, yz, zz.
__host__ __device__ constexpr int sym(int a, int b) { return a == 0 || b == 0 ? a + b : a + b + 1; }

// The unit quaternion of a particle's (w, x, y, z).
__device__ __forceinline__ void unit_quat(const float q[4], double& norm, double h[4]) {
    const double w = q[0], x = q[1], y = q[2], z = q[3];
    norm = sqrt(w * w + x * x + y * y + z * z);
    h[0] = w / norm;
    h[1] = x / norm;
    h[2] = y / norm;
    h[3] = z / norm;
}

// The value through an empty statement that the compiler does not see through: what is
// computed from it later is computed again rather than kept in registers.
__device__ __forceinline__ float reload(float x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Registers: one view (ONE) holds no sums across views and stores its colour gradients before
// the chain rule, so that three waves per SIMD reside; more views need up to 224 registers and
// two. A 1080p view of 1M particles, degree 3: 204 us with 264 registers and one wave, 141 at
// two waves, 134 at three (which spill six registers), 172 at four (which spill more).
template <bool ONE>
constexpr int kAnisoGradWaves = ONE ? 3 : 2;

// One thread per particle of one scene. Per view: the entry records of the particle are
// summed in emit order (FP32, fixed order), turned into the gradients of the footprint
// centre (u, v), the conic (A, B, C), the opacity and the colour, and chained in FP64
// through Sigma_2D = T Sigma T^T (T = J V, eq. 7; conic = Sigma_2D^-1) to the centre and,
// accumulated over the views, to Sigma = R S S^T R^T (eq. 6), hence to the quaternion
// (through its normalisation) and the three scales.
template <int DEG, bool ONE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kAnisoGradWaves<ONE>)))
aniso_grad_project_kernel(const AnisoGradPack pk, const float4* __restrict__ rec,
                                                                 const uint8_t* __restrict__ has_rec,
                                                                 const float4* __restrict__ record,
                                                                 const float2* __restrict__ conic,
                                                                 const uint32_t* __restrict__ tile_count,
                                                                 const uint32_t* __restrict__ offsets,
                                                                 const uint32_t* __restrict__ count_p,
                                                                 const int32_t* __restrict__ status) {
    __shared__ RecShared<kRecVec4<true>> sh;
    if (*status != kStatusOk) return;
    const uint32_t n_entries = *count_p;
    // threads past the last particle stay for the shared record sums, on the last one's inputs
    const bool in = blockIdx.x * 256u + threadIdx.x < pk.n;
    const uint32_t i = min(blockIdx.x * 256u + threadIdx.x, pk.n - 1u);
    const uint32_t n = pk.n;
    constexpr int K = (DEG + 1) * (DEG + 1);
    const float mx = pk.pos[i], my = pk.pos[n + i], mz = pk.pos[2 * n + i];
    const float q4[4] = {pk.rot[i], pk.rot[n + i], pk.rot[2 * n + i], pk.rot[3 * n + i]};
    const float s3[3] = {pk.scale[i], pk.scale[n + i], pk.scale[2 * n + i]};
    // Sigma = R diag(s^2) R^T (symmetric: xx, xy, xz, yy, yz, zz)
    double Sig[6];
    {
        double qn, h[4], Rq[9];
        unit_quat(q4, qn, h);
        quat_rot(h[0], h[1], h[2], h[3], Rq);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                if (b < a) continue;
                double acc = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) acc += Rq[3 * a + c] * (double)s3[c] * (double)s3[c] * Rq[3 * b + c];
                Sig[sym(a, b)] = acc;
            }
    }

    float gmx = 0.0f, gmy = 0.0f, gmz = 0.0f, gop = 0.0f;
    double GS[6];   // dL/dSigma, summed over the views (symmetric)
#pragma unroll
    for (int k = 0; k < 6; ++k) GS[k] = 0.0;
    double gmu64[3] = {0.0, 0.0, 0.0};
    bool any = false;
    float gcol[3 * K];
    float coef[3 * K];
#pragma unroll
    for (int k = 0; k < 3 * K; ++k) {
        gcol[k] = 0.0f;
        coef[k] = pk.color[(size_t)k * n + i];
    }

    RecRun next = record_run(tile_count, offsets, pk.v[0].p_off + i, in, n_entries);
    const int nv = ONE ? 1 : pk.nv;
    for (int vv = 0; vv < nv; ++vv) {
        const GradView& gv = pk.v[vv];
        const uint32_t pi = gv.p_off + i;
        const RecRun cur = next;
        if (vv + 1 < nv) next = record_run(tile_count, offsets, pk.v[vv + 1].p_off + i, in, n_entries);
        float S[12];
        const bool act = sum_records<3>(sh, rec, has_rec, cur.e0, cur.cnt, S) && cur.cnt != 0;
        const float drgb[3] = {S[6], S[7], S[8]};
        if (act) color_backward<DEG>(CoefRef{coef}, drgb, gv.eye, mx, my, mz, gcol, gmx, gmy, gmz);
        // a single view's colour gradients are complete: stored here, they and the coefficients
        // need no registers beside the chain rule below
        if (ONE && in) store_color<K>(pk, i, gcol);
        if (!act) continue;
        any = true;
        gop += S[5];
        const double A = (double)record[2 * (size_t)pi].z;
        const float2 bc = conic[pi];
        const double B = (double)bc.x, C = (double)bc.y;
        // sums k dx, k dy, k dx^2, k dx dy, k dy^2 -> gradients of u, v and the conic
        const double du = 2.0 * (A * S[0] + B * S[1]), dv = 2.0 * (B * S[0] + C * S[1]);
        const double dA = -(double)S[2], dB = -2.0 * (double)S[3], dC = -(double)S[4];
        // dL/dSigma_2D = -Ci Gc Ci, Ci = [[A, B], [B, C]], Gc = [[dA, dB/2], [dB/2, dC]]
        const double m00 = A * dA + B * 0.5 * dB, m01 = A * 0.5 * dB + B * dC;
        const double m10 = B * dA + C * 0.5 * dB, m11 = B * 0.5 * dB + C * dC;
        const double G00 = -(m00 * A + m01 * B), G01 = -(m00 * B + m01 * C), G11 = -(m10 * B + m11 * C);
        // camera-space centre and T = J V
        double V[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) V[k] = (double)gv.R[k];
        const double px = V[0] * mx + V[1] * my + V[2] * mz + (double)gv.t[0];
        const double py = V[3] * mx + V[4] * my + V[5] * mz + (double)gv.t[1];
        const double pz = V[6] * mx + V[7] * my + V[8] * mz + (double)gv.t[2];
        const double f = (double)gv.f, iz = 1.0 / pz;
        const double J00 = f * iz, J02 = -f * px * iz * iz, J12 = -f * py * iz * iz;
        double T[6];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            T[c] = J00 * V[c] + J02 * V[6 + c];
            T[3 + c] = J00 * V[3 + c] + J12 * V[6 + c];
        }
        // dL/dSigma += T^T G T
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b)
                if (b >= a)
                    GS[sym(a, b)] += T[a] * (G00 * T[b] + G01 * T[3 + b]) + T[3 + a] * (G01 * T[b] + G11 * T[3 + b]);
        // dL/dT = 2 G T Sigma, dL/dJ = dL/dT V^T
        double TS[6];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                TS[3 * r + c] = T[3 * r] * Sig[sym(0, c)] + T[3 * r + 1] * Sig[sym(1, c)] + T[3 * r + 2] * Sig[sym(2, c)];
        double GT[6];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            GT[c] = 2.0 * (G00 * TS[c] + G01 * TS[3 + c]);
            GT[3 + c] = 2.0 * (G01 * TS[c] + G11 * TS[3 + c]);
        }
        double GJ[6];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                GJ[3 * r + c] = GT[3 * r] * V[3 * c] + GT[3 * r + 1] * V[3 * c + 1] + GT[3 * r + 2] * V[3 * c + 2];
        // J = [[f/z, 0, -f p_x/z^2], [0, f/z, -f p_y/z^2]]; u = f p_x / z + cx, v likewise
        const double iz2 = iz * iz;
        double dpx = -GJ[2] * f * iz2 + du * f * iz;
        double dpy = -GJ[5] * f * iz2 + dv * f * iz;
        double dpz = -(GJ[0] + GJ[4]) * f * iz2 + 2.0 * f * (GJ[2] * px + GJ[5] * py) * iz2 * iz -
                     (du * f * px + dv * f * py) * iz2;
        gmu64[0] += V[0] * dpx + V[3] * dpy + V[6] * dpz;
        gmu64[1] += V[1] * dpx + V[4] * dpy + V[7] * dpz;
        gmu64[2] += V[2] * dpx + V[5] * dpy + V[8] * dpz;
    }
    float grot[4] = {0.0f, 0.0f, 0.0f, 0.0f}, gsc[3] = {0.0f, 0.0f, 0.0f};
    if (any) {
        const float qr[4] = {reload(q4[0]), reload(q4[1]), reload(q4[2]), reload(q4[3])};
        const double sc[3] = {(double)s3[0], (double)s3[1], (double)s3[2]};
        double qn, h[4], Rq[9];
        unit_quat(qr, qn, h);
        quat_rot(h[0], h[1], h[2], h[3], Rq);
        // Sigma = R diag(s^2) R^T: dL/dR = 2 GS R diag(s^2), dL/ds_b = 2 s_b (R^T GS R)_bb
        double GR[9];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b)
                GR[3 * a + b] = 2.0 * (GS[sym(a, 0)] * Rq[b] + GS[sym(a, 1)] * Rq[3 + b] + GS[sym(a, 2)] * Rq[6 + b]) *
                                sc[b] * sc[b];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            double acc = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int c = 0; c < 3; ++c) acc += Rq[3 * a + b] * GS[sym(a, c)] * Rq[3 * c + b];
            gsc[b] = (float)(2.0 * sc[b] * acc);
        }
        // dR/d(w, x, y, z) of the rotation formula, at the unit quaternion
        const double w = h[0], x = h[1], y = h[2], z = h[3];
        const double dRw[9] = {0.0, -2 * z, 2 * y, 2 * z, 0.0, -2 * x, -2 * y, 2 * x, 0.0};
        const double dRx[9] = {0.0, 2 * y, 2 * z, 2 * y, -4 * x, -2 * w, 2 * z, 2 * w, -4 * x};
        const double dRy[9] = {-4 * y, 2 * x, 2 * w, 2 * x, 0.0, 2 * z, -2 * w, 2 * z, -4 * y};
        const double dRz[9] = {-4 * z, -2 * w, 2 * x, 2 * w, -4 * z, 2 * y, 2 * x, 2 * y, 0.0};
        double dq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            dq[0] += GR[k] * dRw[k];
            dq[1] += GR[k] * dRx[k];
            dq[2] += GR[k] * dRy[k];
            dq[3] += GR[k] * dRz[k];
        }
        // through the normalisation q / |q|
        const double radial = h[0] * dq[0] + h[1] * dq[1] + h[2] * dq[2] + h[3] * dq[3];
#pragma unroll
        for (int k = 0; k < 4; ++k) grot[k] = (float)((dq[k] - h[k] * radial) / qn);
        gmx += (float)gmu64[0];
        gmy += (float)gmu64[1];
        gmz += (float)gmu64[2];
    }
    if (!in) return;
    if (!ONE) store_color<K>(pk, i, gcol);
    const float gmu[3] = {gmx, gmy, gmz};
    if (pk.accumulate) {
#pragma unroll
        for (int k = 0; k < 3; ++k) pk.g_pos[(size_t)k * n + i] += gmu[k];
#pragma unroll
        for (int k = 0; k < 4; ++k) pk.g_rot[(size_t)k * n + i] += grot[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) pk.g_scale[(size_t)k * n + i] += gsc[k];
        pk.g_opacity[i] += gop;
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) pk.g_pos[(size_t)k * n + i] = gmu[k];
#pragma unroll
        for (int k = 0; k < 4; ++k) pk.g_rot[(size_t)k * n + i] = grot[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) pk.g_scale[(size_t)k * n + i] = gsc[k];
        pk.g_opacity[i] = gop;
    }
}

// The kernels of degrees 0 to 3.
template <bool ONE>
static std::array<decltype(&aniso_grad_project_kernel<0, ONE>), 4> aniso_grad_kernels() {
    return {aniso_grad_project_kernel<0, ONE>, aniso_grad_project_kernel<1, ONE>, aniso_grad_project_kernel<2, ONE>,
            aniso_grad_project_kernel<3, ONE>};
}

static size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

// Workspace: gradient records (32 B per entry of capacity, 48 B for the anisotropic
// family) and their marks (1 B per entry), the tile queue, the chunk item count and the chunk items (two words each; at
// most capacity / kCkptChunk + tiles).
static size_t bwd_heavy_items(uint64_t capacity, uint32_t tiles) {
    return (size_t)(capacity / kCkptChunk) + tiles + 1;
}

static size_t rec_bytes(bool an) { return an ? 48 : 32; }

size_t render_bwd_ws(uint64_t capacity, const isogs_camera* cams, int32_t nv, bool an) {
    const uint32_t tiles = max_group_tiles(cams, nv);
    return round256((size_t)capacity * rec_bytes(an)) + round256((size_t)capacity) +
           round256(tile_queue_words(tiles) * 4) + 256 + bwd_heavy_items(capacity, tiles) * 8 + 256;
}

// Reverse compositing of every view into the entry records (both families): chunks of
// long tiles (with checkpoints), then tiles longest first. Returns the records (rec NULL: a
// launch failed).
struct BwdRecords {
    float4* rec;
    uint8_t* has_rec;
};

static BwdRecords launch_composite_bwd(bool an, const int32_t* n_all, const isogs_camera* cams, int32_t nv,
                                    const isogs_projected* proj, const float* conic, const isogs_bins* bins,
                                    const float* bg, const float* image, const float* dL_dimage,
                                    const float* T_final, const uint32_t* n_last, const float* ckpt, void* ws,
                                    hipStream_t stream) {
    const uint32_t max_tiles = max_group_tiles(cams, nv);
    char* base = static_cast<char*>(ws);
    float4* rec = reinterpret_cast<float4*>(base);
    base += round256((size_t)bins->capacity * rec_bytes(an));
    uint8_t* has_rec = reinterpret_cast<uint8_t*>(base);
    base += round256((size_t)bins->capacity);
    uint32_t* q = reinterpret_cast<uint32_t*>(base);
    base += round256(tile_queue_words(max_tiles) * 4);
    uint32_t* heavy_count = reinterpret_cast<uint32_t*>(base);
    uint32_t* heavy = reinterpret_cast<uint32_t*>(base + 256);
    const uint32_t heavy_max = (uint32_t)bwd_heavy_items(bins->capacity, max_tiles);
    // a long tile of len entries has ceil(len / kCkptChunk) chunks, at most len / kCkptChunk
    // more items than tiles; over ranges that partition the entries, at most
    // capacity / kCkptChunk more in all
    const uint32_t extra_items = ckpt ? (uint32_t)(bins->capacity / kCkptChunk) + 1u : 0u;
    if (bins->capacity)
        hipLaunchKernelGGL(clear_marks_kernel, dim3((unsigned)std::min<uint64_t>(2048, (bins->capacity + 4095) / 4096)),
                           dim3(256), 0, stream, has_rec, bins->count, bins->capacity);
    uint32_t p_off = 0, tile_base = 0, pix_off = 0;
    for (int v0 = 0; v0 < nv; v0 += kMaxViews) {
        const int m = min(kMaxViews, nv - v0);
        RenderPack pk{};
        uint32_t blocks;
        const uint32_t tile0 = tile_base;
        fill_render_pack(pk, cams + v0, n_all + v0, 0, m, p_off, tile_base, pix_off, blocks);
        set_render_limits(pk, n_all, nv, bins->capacity);
        if (!blocks) continue;
        uint32_t* order = launch_tile_queue(q, bins->ranges, tile0, blocks, pk.n_entries_cap, stream);
        if (ckpt) {
            hipLaunchKernelGGL(fill_u32_kernel_b, dim3(1), dim3(64), 0, stream, heavy_count, 1u);
            hipLaunchKernelGGL(bwd_chunk_list_kernel, dim3((blocks + kReachTiles - 1) / kReachTiles), dim3(256), 0,
                               stream, pk, bins->ranges, tile0, blocks, n_last, bins->status, heavy, heavy_count,
                               heavy_max);
        }
        const BwdArgs a{reinterpret_cast<const float4*>(proj->record), reinterpret_cast<const float2*>(conic),
                        bins->pidx, bins->offsets, bins->ranges, bins->status, bg[0], bg[1], bg[2], image, dL_dimage,
                        T_final, n_last, reinterpret_cast<const float4*>(ckpt), rec, has_rec, order, q, blocks, heavy,
                        heavy_count, heavy_max};
        const uint32_t items = blocks + extra_items;
        const bool loop = items > kBwdLoopItems;
        auto k = an ? (loop ? aniso_bwd_ordered_kernel<true> : aniso_bwd_ordered_kernel<false>)
                    : (loop ? composite_bwd_ordered_kernel<true> : composite_bwd_ordered_kernel<false>);
        hipLaunchKernelGGL(k, dim3(loop ? kBwdLoopGrid : items), dim3(256), 0, stream, pk, a);
        if (hipPeekAtLastError() != hipSuccess) return {nullptr, nullptr};
    }
    return {rec, has_rec};
}

// Views grouped by scene (equal position buffers), in view order; calls fn(first view of
// the scene, views[], count) for each scene.
template <typename Fn>
static void for_each_scene(const float* const* pos, int32_t nv, Fn fn) {
    bool handled[4096] = {false};
    for (int v = 0; v < nv; ++v) {
        if (handled[v]) continue;
        int pending[4096];
        int np = 0;
        for (int u = v; u < nv; ++u)
            if (!handled[u] && pos[u] == pos[v]) {
                handled[u] = true;
                pending[np++] = u;
            }
        fn(v, pending, np);
    }
}

static void fill_grad_view(GradView& g, const isogs_camera& c, uint32_t p_off) {
    g.p_off = p_off;
    for (int k = 0; k < 9; ++k) g.R[k] = c.R[k];
    for (int k = 0; k < 3; ++k) g.t[k] = c.t[k], g.eye[k] = c.eye[k];
    g.f = c.f;
    g.cx = c.cx;
    g.cy = c.cy;
}

int launch_render_bwd(const isogs_scene* scenes, const isogs_camera* cams, int32_t nv,
                      const isogs_projected* proj, const isogs_bins* bins, const float* bg,
                      const float* image, const float* dL_dimage, const float* T_final, const uint32_t* n_last,
                      const float* ckpt, const isogs_scene* grads, void* ws, hipStream_t stream) {
    if (nv > 4096) return -1;
    int32_t n_all[4096];
    uint32_t view_off[4096];
    const float* pos[4096];
    uint32_t o = 0;
    for (int v = 0; v < nv; ++v) {
        n_all[v] = scenes[v].n;
        view_off[v] = o;
        o += (uint32_t)scenes[v].n;
        pos[v] = scenes[v].pos;
    }
    // 1. reverse compositing
    const BwdRecords br = launch_composite_bwd(false, n_all, cams, nv, proj, nullptr, bins, bg, image, dL_dimage, T_final,
                                             n_last, ckpt, ws, stream);
    if (!br.rec) return -1;
    // 2. per scene: reduce records over its views (in view order) and chain to parameters
    int rc = 0;
    for_each_scene(pos, nv, [&](int v, const int* pending, int np) {
        const isogs_scene& sc = scenes[v];
        const isogs_scene& gs = grads[v];
        for (int b0 = 0; b0 < np && !rc; b0 += kMaxViews) {
            GradPack gp{};
            gp.nv = min(kMaxViews, np - b0);
            gp.accumulate = b0 > 0;
            gp.pos = sc.pos;
            gp.scale = sc.scale;
            gp.opacity = sc.opacity;
            gp.color = sc.color;
            gp.n = (uint32_t)sc.n;
            gp.sh_degree = sc.sh_degree;
            gp.g_pos = const_cast<float*>(gs.pos);
            gp.g_scale = const_cast<float*>(gs.scale);
            gp.g_opacity = const_cast<float*>(gs.opacity);
            gp.g_color = const_cast<float*>(gs.color);
            for (int j = 0; j < gp.nv; ++j) fill_grad_view(gp.v[j], cams[pending[b0 + j]], view_off[pending[b0 + j]]);
            if (sc.n > 0) {
                const dim3 grid((sc.n + 255) / 256);
                switch (sc.sh_degree) {
                    case 0: hipLaunchKernelGGL(grad_project_kernel<0>, grid, dim3(256), 0, stream, gp, br.rec, br.has_rec, proj->tile_count, bins->offsets, bins->count, bins->status); break;
                    case 1: hipLaunchKernelGGL(grad_project_kernel<1>, grid, dim3(256), 0, stream, gp, br.rec, br.has_rec, proj->tile_count, bins->offsets, bins->count, bins->status); break;
                    case 2: hipLaunchKernelGGL(grad_project_kernel<2>, grid, dim3(256), 0, stream, gp, br.rec, br.has_rec, proj->tile_count, bins->offsets, bins->count, bins->status); break;
                    default: hipLaunchKernelGGL(grad_project_kernel<3>, grid, dim3(256), 0, stream, gp, br.rec, br.has_rec, proj->tile_count, bins->offsets, bins->count, bins->status); break;
                }
            }
            if (hipPeekAtLastError() != hipSuccess) rc = -1;
        }
    });
    return rc;
}

int launch_aniso_render_bwd(const isogs_aniso_scene* scenes, const isogs_camera* cams, int32_t nv,
                            const isogs_aniso_projected* proj, const isogs_bins* bins, const float* bg,
                            const float* image, const float* dL_dimage, const float* T_final,
                            const uint32_t* n_last, const float* ckpt, const isogs_aniso_scene* grads, void* ws,
                            hipStream_t stream) {
    if (nv > 4096) return -1;
    int32_t n_all[4096];
    uint32_t view_off[4096];
    const float* pos[4096];
    uint32_t o = 0;
    for (int v = 0; v < nv; ++v) {
        n_all[v] = scenes[v].n;
        view_off[v] = o;
        o += (uint32_t)scenes[v].n;
        pos[v] = scenes[v].pos;
    }
    const BwdRecords br = launch_composite_bwd(true, n_all, cams, nv, &proj->fp, proj->conic, bins, bg, image, dL_dimage,
                                             T_final, n_last, ckpt, ws, stream);
    if (!br.rec) return -1;
    int rc = 0;
    for_each_scene(pos, nv, [&](int v, const int* pending, int np) {
        const isogs_aniso_scene& sc = scenes[v];
        const isogs_aniso_scene& gs = grads[v];
        for (int b0 = 0; b0 < np && !rc; b0 += kMaxViews) {
            AnisoGradPack gp{};
            gp.nv = min(kMaxViews, np - b0);
            gp.accumulate = b0 > 0;
            gp.pos = sc.pos;
            gp.rot = sc.rot;
            gp.scale = sc.scale;
            gp.opacity = sc.opacity;
            gp.color = sc.color;
            gp.n = (uint32_t)sc.n;
            gp.sh_degree = sc.sh_degree;
            gp.g_pos = const_cast<float*>(gs.pos);
            gp.g_rot = const_cast<float*>(gs.rot);
            gp.g_scale = const_cast<float*>(gs.scale);
            gp.g_opacity = const_cast<float*>(gs.opacity);
            gp.g_color = const_cast<float*>(gs.color);
            for (int j = 0; j < gp.nv; ++j) fill_grad_view(gp.v[j], cams[pending[b0 + j]], view_off[pending[b0 + j]]);
            if (sc.n > 0) {
                const dim3 grid((sc.n + 255) / 256);
                const float4* r = reinterpret_cast<const float4*>(proj->fp.record);
                const float2* k = reinterpret_cast<const float2*>(proj->conic);
                const uint32_t* tc = proj->fp.tile_count;
                const auto kernels = gp.nv == 1 ? aniso_grad_kernels<true>() : aniso_grad_kernels<false>();
                hipLaunchKernelGGL(kernels[sc.sh_degree < 3 ? sc.sh_degree : 3], grid, dim3(256), 0, stream, gp, br.rec,
                                   br.has_rec, r, k, tc, bins->offsets, bins->count, bins->status);
            }
            if (hipPeekAtLastError() != hipSuccess) rc = -1;
        }
    });
    return rc;
}

}  // namespace isogs
