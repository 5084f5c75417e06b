// Tile binning: per-(frame, tile) Gaussian lists in depth order, built from
// the frame-major depth-sorted items without sorting (tile, Gaussian) pairs.
//
// The compositing loop of paper §3 walks, for every pixel, the Gaussians of
// its tile front to back.  Each item (frame, Gaussian) covers a rectangle of
// tiles; its entry for tile t sits at start[t] + (number of items before it
// in depth order that cover t).  Two levels:
//
// Level A -- items into groups of 8x8 tiles.  The depth-ordered items of a
//   frame are cut into chunks: per-chunk group counts (LDS), a column scan
//   over the chunks, an exclusive scan over (frame, group), then one wave per
//   chunk places 64 items at a time, every lane at once: the lanes that share
//   a group come from four ballot masks (by group column and row), and a
//   lane's rank among them is its offset in that group's list.
// Level B -- the tile lists' lengths.  Each group list is cut into segments; a
//   counting pass (an 8x8 difference array per wave) and an exclusive scan
//   over (frame, tile) give every tile's length and its place in the pair
//   array.  The lists themselves are not placed: the forward composite filters
//   its tile's entries out of the group list as far as it goes (walk.h), and
//   writes down that part for the backward.  An opaque tile ends after a few
//   hundred of its entries (1M x 16 frames: 150 of 14000), so placing all of
//   them was 1.44 of 6.5 ms there and 55 of 880 us at 200k x 8, against 8 and
//   5 us more in the composite; where no tile ends early (600k Gaussians of 1
//   to 2 pixels) the filter costs about what the placement did.
#include "block_scan.h"
#include "common.h"
#include "walk.h"

namespace gft {

namespace {

__device__ __forceinline__ void unpack_rect(uint2 rc, uint32_t& xlo, uint32_t& xhi, uint32_t& ylo,
                                            uint32_t& yhi) {
    xlo = rc.x & 0xffff;
    xhi = rc.x >> 16;
    ylo = rc.y & 0xffff;
    yhi = rc.y >> 16;
}

struct Groups {
    int ngx, ngy, ng;   // groups per row, per column, per frame
};

__device__ __forceinline__ Groups groups_of(const Params& P) {
    Groups g;
    g.ngx = (P.ntx + kGroupW - 1) / kGroupW;
    g.ngy = (P.nty + kGroupH - 1) / kGroupH;
    g.ng = g.ngx * g.ngy;
    return g;
}

// The depth-sorted items: in buffer 1, or in buffer 0 where the sort needed
// its fourth pass.
struct DepthOrder {
    const uint32_t *key0, *key1, *item0, *item1;
    const uint2 *rect0, *rect1;
    const uint32_t* flag;
    __device__ __forceinline__ bool wide() const { return *flag != 0u; }
    __device__ __forceinline__ const uint32_t* keys(bool w) const { return w ? key0 : key1; }
    __device__ __forceinline__ const uint32_t* items(bool w) const { return w ? item0 : item1; }
    __device__ __forceinline__ const uint2* rects(bool w) const { return w ? rect0 : rect1; }
};
DepthOrder depth_order(const Workspace& w) {
    return {w.dkey[0], w.dkey[1], w.dval[0], w.dval[1], w.drect[0], w.drect[1], w.sctl + kSortWide};
}

// ---- level A: items -> groups ----------------------------------------------

// Group counts of each chunk of C items: one workgroup of 256 threads per CPW
// chunks (CPW = 512 / C, between 1 and 4, so that every thread counts two or
// more items and short chunks do not each pay a workgroup launch).
constexpr int kMaxChunksPerBlock = 4;

__global__ void __launch_bounds__(256) k_group_count(Params P, int C, int QC, int CPW,
                                                     DepthOrder order,
                                                     uint32_t* __restrict__ cntA, uint32_t* __restrict__ touch) {
    // no item has been walked yet (the flags' bytes, four at a time; the
    // workspace pads them to whole words)
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < (P.n * P.F + 3) / 4; i += (int64_t)gridDim.x * 256)
        touch[i] = 0u;
    __shared__ uint32_t lcnt[kMaxChunksPerBlock][kMaxGroupsPerFrame];
    const bool wide = order.wide();
    const uint32_t* dkey = order.keys(wide);
    const uint2* drect = order.rects(wide);
    const Groups G = groups_of(P);
    const int TPC = 256 / CPW;   // threads per chunk
    const int sub = (int)threadIdx.x / TPC, lt = (int)threadIdx.x - sub * TPC;
    const int chunk = blockIdx.x * CPW + sub;
    const bool have = chunk < P.F * QC;
    uint32_t* cnt = lcnt[sub];
    for (int t = lt; t < G.ng; t += TPC) cnt[t] = 0;
    __syncthreads();
    if (have) {
        const int f = chunk / QC, q = chunk - f * QC;
        const long long beg = (long long)f * P.n + (long long)q * C;
        const long long end = min(beg + C, (long long)(f + 1) * P.n);
        for (long long j = beg + lt; j < end; j += TPC) {
            if (dkey[j] == kCulledKey) continue;
            uint32_t xlo, xhi, ylo, yhi;
            unpack_rect(drect[j], xlo, xhi, ylo, yhi);
            for (uint32_t gy = ylo / kGroupH; gy <= yhi / kGroupH; ++gy)
                for (uint32_t gx = xlo / kGroupW; gx <= xhi / kGroupW; ++gx)
                    atomicAdd(&cnt[gy * G.ngx + gx], 1u);
        }
    }
    __syncthreads();
    if (have) {
        uint32_t* out = cntA + (size_t)chunk * G.ng;
        for (int t = lt; t < G.ng; t += TPC) out[t] = cnt[t];
    }
}

// grid (ng, F), 256 threads: one workgroup per (frame, group) column.
// Exclusive scan of the column over the chunks of its frame (each thread a
// run of consecutive chunks), and the column total; the tile counts of the
// group are cleared for k_tile_count.
__global__ void __launch_bounds__(256) k_group_colscan(Params P, int QC, uint32_t* __restrict__ cntA,
                                                       uint32_t* __restrict__ lenA, uint32_t* __restrict__ tcount) {
    __shared__ uint32_t scratch[8];
    const Groups G = groups_of(P);
    const int gi = blockIdx.x, f = blockIdx.y;
    if (threadIdx.x < kGroupW * kGroupH) {   // the group's tile counts start at 0
        const int tx = gi % G.ngx * kGroupW + threadIdx.x % kGroupW, ty = gi / G.ngx * kGroupH + threadIdx.x / kGroupW;
        if (tx < P.ntx && ty < P.nty) tcount[(size_t)f * P.n_tiles + ty * P.ntx + tx] = 0u;
    }
    const int per = (QC + 255) / 256;
    const int q0 = min((int)threadIdx.x * per, QC), q1 = min(q0 + per, QC);
    uint32_t* col = cntA + (size_t)f * QC * G.ng + gi;
    // 8 loads in flight per round (a thread's run is 4-8 chunks at 1.6M-16M
    // items)
    uint32_t s = 0;
    for (int q = q0; q < q1; q += 8) {
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = q + i < q1 ? col[(size_t)(q + i) * G.ng] : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) s += v[i];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan<uint32_t, 256>(s, scratch, &total);
    for (int q = q0; q < q1; q += 8) {
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = q + i < q1 ? col[(size_t)(q + i) * G.ng] : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (q + i < q1) col[(size_t)(q + i) * G.ng] = run;
            run += v[i];
        }
    }
    if (threadIdx.x == 0) lenA[(size_t)f * G.ng + gi] = total;
}

// Single workgroup: group-list ranges (exclusive scan of the lengths) and the
// first level-B segment of every group.  The level-A lists are bounded by the
// pair capacity (every group entry yields at least one pair).
__global__ void __launch_bounds__(1024) k_group_scan(const uint32_t* __restrict__ lenA, int K, int S,
                                                     unsigned long long cap, uint2* __restrict__ granges,
                                                     uint32_t* __restrict__ seg_start) {
    __shared__ unsigned long long scratch[17];
    __shared__ uint32_t scratch32[17];
    unsigned long long carry = 0;
    uint32_t scarry = 0;
    for (int base = 0; base < K; base += 1024) {
        const int i = base + threadIdx.x;
        const unsigned long long v = i < K ? lenA[i] : 0ull;
        unsigned long long tot;
        uint32_t stot;
        const unsigned long long ex = block_exclusive_scan<unsigned long long, 1024>(v, scratch, &tot);
        const unsigned long long a = carry + ex, b = a + v;
        const unsigned long long ac = a < cap ? a : cap, bc = b < cap ? b : cap;
        // segments of the stored part of the list only (the lists are cut at
        // the capacity)
        const uint32_t nsg = (uint32_t)((bc - ac + S - 1) / S);
        const uint32_t sex = block_exclusive_scan<uint32_t, 1024>(nsg, scratch32, &stot);
        if (i < K) {
            granges[i] = make_uint2((uint32_t)ac, (uint32_t)bc);
            seg_start[i] = scarry + sex;
        }
        carry += tot;
        scarry += stot;
    }
    if (threadIdx.x == 0) seg_start[K] = scarry;
}

// Placing pass of level A.  Work item = (run of RA consecutive chunks of one
// frame, group row gy); one wave walks the run's depth-ordered items 64 at a
// time (lane = item) and, for each group column, ballots the lanes whose
// rectangle covers that group: each writes at the group's cursor plus its
// rank among them, so one store appends a contiguous run to the group list
// and depth order holds inside every list.  A wave appends each group's run
// over the whole run of chunks, so its stores fill whole cache lines instead
// of scattering a few entries per group and batch.
// FAST: the row's group lists all end strictly below the capacity (their
// ranges are clamped to it), so the stores need no check.  REG: the row has
// at most kGroupW groups, whose cursors stay in scalar registers under an
// unrolled, branch-free column loop (an empty ballot stores nothing);
// otherwise they live in LDS.  NB: runs of at least 16 batches load 8
// batches at a time (fewer waits per run); shorter runs load each batch
// while the previous one is placed (measured faster there).
template <bool FAST, bool REG, int NB>
__device__ __forceinline__ void place_group_row(const Groups& G, long long beg, long long end, uint32_t gy, int lane,
                                                uint32_t* cursor, uint32_t (&cur)[kGroupW], uint32_t cap,
                                                const uint32_t* __restrict__ dval,
                                                const uint32_t* __restrict__ dkey,
                                                const uint2* __restrict__ drect,
                                                uint32_t* __restrict__ gval, uint16_t* __restrict__ gloc) {
    const uint32_t oy = gy * kGroupH;
    // one batch: lane = item, covering the groups gx0 .. gx1 of the row
    auto place_batch_a = [&](uint32_t key, uint32_t item, uint2 rect) {
        int gx0 = 1, gx1 = 0;   // empty: never in a ballot
        uint32_t xlo = 0, xhi = 0, ylo = 0, yhi = 0;
        if (key != kCulledKey) {
            unpack_rect(rect, xlo, xhi, ylo, yhi);
            if (ylo / kGroupH <= gy && gy <= yhi / kGroupH) {
                gx0 = (int)(xlo / kGroupW);
                gx1 = (int)(xhi / kGroupW);
            }
        }
        // the rows of the rectangle clipped to this group row
        const uint32_t y0 = max(ylo, oy) - oy, y1 = min(yhi, oy + kGroupH - 1) - oy;
        const uint32_t ybits = pack_rect(0, 7, y0, y1);
        auto place = [&](int c, uint32_t at, uint64_t peers, bool mine) {
            if (mine) {
                const uint32_t pos = at + rank_below(peers);
                const uint32_t ox = (uint32_t)c * kGroupW;
                const uint32_t x0 = max(xlo, ox) - ox, x1 = min(xhi, ox + kGroupW - 1) - ox;
                if (FAST || pos < cap) {
                    gval[pos] = item;
                    gloc[pos] = (uint16_t)(pack_rect(x0, x1, 0, 7) | ybits);
                }
            }
        };
        if constexpr (REG) {
#pragma unroll
            for (int c = 0; c < kGroupW; ++c) {   // columns past the frame never match
                const bool mine = gx0 <= c && c <= gx1;
                const uint64_t peers = __ballot(mine);
                place(c, cur[c], peers, mine);
                cur[c] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(cur[c] + (uint32_t)__popcll(peers)));
            }
        } else {
            for (int c = 0; c < G.ngx; ++c) {
                const bool mine = gx0 <= c && c <= gx1;
                const uint64_t peers = __ballot(mine);
                if (peers == 0ull) continue;
                const uint32_t at = cursor[c];
                place(c, at, peers, mine);
                if (lane == 0) cursor[c] = at + (uint32_t)__popcll(peers);
            }
            // lane 0's cursor writes precede the next batch's reads by every lane
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };
    if constexpr (NB == 1) {
        // the next batch's key, item and rectangle are loaded while this
        // batch is placed
        uint32_t nkey = kCulledKey, nitem = 0;
        uint2 nrect = make_uint2(0u, 0u);
        if (beg + lane < end) {
            nkey = dkey[beg + lane];
            nitem = dval[beg + lane];
            nrect = drect[beg + lane];
        }
        for (long long j0 = beg; j0 < end; j0 += 64) {
            const uint32_t key = nkey, item = nitem;
            const uint2 rect = nrect;
            const long long jn = j0 + 64 + lane;
            nkey = kCulledKey;
            if (jn < end) {
                nkey = dkey[jn];
                nitem = dval[jn];
                nrect = drect[jn];
            }
            place_batch_a(key, item, rect);
        }
    } else {
        // NB batches at a time, all their loads in flight before the first
        // of them is placed
        for (long long r0 = beg; r0 < end; r0 += 64 * NB) {
            uint32_t bkey[NB], bitem[NB];
            uint2 brect[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const long long j = r0 + 64 * b + lane;
                bkey[b] = kCulledKey;
                bitem[b] = 0;
                brect[b] = make_uint2(0u, 0u);
                if (j < end) {
                    bkey[b] = dkey[j];
                    bitem[b] = dval[j];
                    brect[b] = drect[j];
                }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (r0 + 64 * b >= end) break;   // wave-uniform
                place_batch_a(bkey[b], bitem[b], brect[b]);
            }
        }
    }
}

template <int NB>
__global__ void __launch_bounds__(64) k_group_place(Params P, int C, int QC, int RA,
                                                         DepthOrder order,
                                                         const uint32_t* __restrict__ cntA,
                                                         const uint2* __restrict__ granges,
                                                         uint32_t* __restrict__ gval,
                                                         uint16_t* __restrict__ gloc) {
    extern __shared__ uint32_t cursor[];   // [ngx] list cursors of the work item's group row
    const Groups G = groups_of(P);
    const bool wide = order.wide();
    const uint32_t *dkey = order.keys(wide), *dval = order.items(wide);
    const uint2* drect = order.rects(wide);
    const int lane = threadIdx.x;
    const uint32_t cap = (uint32_t)(P.cap < 0xffffffffull ? P.cap : 0xffffffffull);
    const uint32_t nrun = ((uint32_t)QC + (uint32_t)RA - 1) / (uint32_t)RA;   // runs of RA chunks per frame
    const uint32_t nitems = (uint32_t)P.F * nrun * (uint32_t)G.ngy;
    // the rows of one run are consecutive work items, so they read the run's
    // items through one L2; each XCD takes one contiguous eighth of the work
    // items
    const uint32_t per_xcd = gridDim.x / kXcds, xcd = blockIdx.x % kXcds;
    const uint32_t hi = (uint32_t)((uint64_t)nitems * (xcd + 1) / kXcds);
    for (uint32_t wi = (uint32_t)((uint64_t)nitems * xcd / kXcds) + blockIdx.x / kXcds; wi < hi; wi += per_xcd) {
        const uint32_t fr = wi / (uint32_t)G.ngy;
        const uint32_t gy = wi - fr * (uint32_t)G.ngy;
        const uint32_t f = fr / nrun, q = (fr - f * nrun) * (uint32_t)RA;   // the run's first chunk
        const uint32_t chunk = f * (uint32_t)QC + q;
        const long long beg = (long long)f * P.n + (long long)q * C;
        const long long end = min(beg + (long long)RA * C, (long long)(f + 1) * P.n);
        // cursors: the group list start plus the items of earlier chunks
        const size_t g0 = (size_t)f * G.ng + (size_t)gy * G.ngx;
        const uint32_t* pre = cntA + (size_t)chunk * G.ng + (size_t)gy * G.ngx;
        uint32_t el = 0;
        uint32_t cur[kGroupW];
        // the ranges are clamped to the capacity, so only an end strictly
        // below it proves that the whole list fits
        if (G.ngx <= kGroupW) {   // cursors of lanes 0 .. ngx-1, then wave-uniform
            uint32_t cl = 0;
            if (lane < G.ngx) {
                const uint2 gr = granges[g0 + lane];
                cl = gr.x + pre[lane];
                el = gr.y;
            }
#pragma unroll
            for (int c = 0; c < kGroupW; ++c) cur[c] = (uint32_t)__builtin_amdgcn_readlane((int)cl, c);
            if (__ballot(el >= cap) == 0ull)
                place_group_row<true, true, NB>(G, beg, end, gy, lane, cursor, cur, cap, dval, dkey, drect, gval, gloc);
            else
                place_group_row<false, true, NB>(G, beg, end, gy, lane, cursor, cur, cap, dval, dkey, drect, gval, gloc);
            continue;
        }
        __syncthreads();   // the previous work item's cursor reads are done
        for (int c = lane; c < G.ngx; c += 64) {
            const uint2 gr = granges[g0 + c];
            cursor[c] = gr.x + pre[c];
            el = max(el, gr.y);
        }
        __syncthreads();
        if (__ballot(el >= cap) == 0ull)
            place_group_row<true, false, NB>(G, beg, end, gy, lane, cursor, cur, cap, dval, dkey, drect, gval, gloc);
        else
            place_group_row<false, false, NB>(G, beg, end, gy, lane, cursor, cur, cap, dval, dkey, drect, gval, gloc);
    }
}

// ---- level B: group lists -> tile lists ----------------------------------------

// Largest i in [0, K) with a[i] <= v, for a nondecreasing a with a[0] <= v.
__device__ __forceinline__ int last_le(const uint32_t* __restrict__ a, int K, uint32_t v) {
    int lo = 0, hi = K;   // a[lo] <= v < a[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] <= v) lo = mid; else hi = mid;
    }
    return lo;
}

// Segments (of 128 entries) a wave counts at least, so that the global counts
// take one atomic per tile and 1024 entries, and the entries a lane has in
// flight.
constexpr int kCountRun = 8, kCountLoads = 8;

// Counting pass: entries of each tile's list, added to tcount (cleared by
// k_group_colscan).  Every entry adds the four corners of its rectangle to an
// 8x8 difference array in LDS; a 2-D prefix sum across the lanes turns it into
// per-tile counts, once per group that a wave's run of segments meets.
__global__ void __launch_bounds__(64) k_tile_count(Params P, int S, const uint32_t* __restrict__ seg_start,
                                                   const uint2* __restrict__ granges,
                                                   const uint16_t* __restrict__ gloc,
                                                   uint32_t* __restrict__ tcount) {
    __shared__ int diff[64];
    const Groups G = groups_of(P);
    const int K = P.F * G.ng;
    const uint32_t nseg = seg_start[K];
    const int lane = threadIdx.x;
    // each wave counts a run of consecutive segments: one search for the
    // group of the first, then the group advances with the segments (groups
    // with empty lists have no segments and are stepped over)
    const uint32_t per = max((uint32_t)kCountRun, (nseg + gridDim.x - 1) / gridDim.x);
    const uint32_t b0 = min(blockIdx.x * per, nseg), b1 = min(b0 + per, nseg);
    int fg = b0 < b1 ? last_le(seg_start, K, b0) : 0;
    for (uint32_t b = b0; b < b1;) {
        while (seg_start[fg + 1] <= b) ++fg;
        const uint32_t be = min(seg_start[fg + 1], b1);   // the run's segments of this group
        const uint2 gr = granges[fg];
        const uint32_t beg = gr.x + (b - seg_start[fg]) * (uint32_t)S;
        const uint32_t end = min(beg + (be - b) * (uint32_t)S, gr.y);
        diff[lane] = 0;
        __syncthreads();
        for (uint32_t j0 = beg + lane; j0 < end; j0 += 64 * kCountLoads) {
            uint32_t loc[kCountLoads];
#pragma unroll
            for (int q = 0; q < kCountLoads; ++q) loc[q] = j0 + 64 * q < end ? gloc[j0 + 64 * q] : kEmptyRect;
#pragma unroll
            for (int q = 0; q < kCountLoads; ++q) {
                if (loc[q] == kEmptyRect) continue;
                const LocalRect r = local_rect(loc[q]);
                const bool xin = r.x1 + 1 < (uint32_t)kGroupW, yin = r.y1 + 1 < (uint32_t)kGroupH;
                atomicAdd(&diff[r.y0 * kGroupW + r.x0], 1);
                if (xin) atomicAdd(&diff[r.y0 * kGroupW + r.x1 + 1], -1);
                if (yin) atomicAdd(&diff[(r.y1 + 1) * kGroupW + r.x0], -1);
                if (xin && yin) atomicAdd(&diff[(r.y1 + 1) * kGroupW + r.x1 + 1], 1);
            }
        }
        __syncthreads();
        int v = diff[lane];
        for (int d = 1; d < kGroupW; d <<= 1) {
            const int u = __shfl_up(v, d, 64);
            if (lane % kGroupW >= d) v += u;
        }
        for (int d = kGroupW; d < 64; d <<= 1) {
            const int u = __shfl_up(v, d, 64);
            if (lane >= d) v += u;
        }
        const int f = fg / G.ng, gi = fg - f * G.ng;
        const uint32_t gy = gi / G.ngx, gx = gi - gy * G.ngx;
        const uint32_t tx = gx * kGroupW + lane % kGroupW, ty = gy * kGroupH + lane / kGroupW;
        if (v != 0 && tx < (uint32_t)P.ntx && ty < (uint32_t)P.nty)
            atomicAdd(&tcount[(size_t)f * P.n_tiles + ty * P.ntx + tx], (uint32_t)v);
        __syncthreads();   // diff is cleared for the next group
        b = be;
    }
}

// Introspection: the whole list of every tile (one wave each).  The forward
// itself writes only the part of a list that it composites.
__global__ void __launch_bounds__(64) k_tile_lists(Params P, const uint2* __restrict__ ranges,
                                                   const uint2* __restrict__ granges,
                                                   const uint32_t* __restrict__ gval,
                                                   const uint16_t* __restrict__ gloc,
                                                   uint32_t* __restrict__ tval) {
    const int w = blockIdx.x, lane = threadIdx.x;
    const int f = w / P.n_tiles, tile = w - f * P.n_tiles;
    const int ty = tile / P.ntx, tx = tile - ty * P.ntx;
    const uint2 rg = ranges[w];
    if (rg.x == rg.y) return;
    uint32_t at = rg.x;
    TileWalk<1> walk = tile_walk<1>(P, f, tx, ty, granges, gloc, 0, lane);
    while (walk.more() && at < rg.y) {
        const TileWalk<1>::Hits h = walk.round();
        h.each([&](uint32_t entry, uint32_t pos) {
            if (at + pos < rg.y) tval[at + pos] = gval[entry];
        });
        at += h.count();
    }
}

// Single workgroup: tile-list ranges = exclusive scan of the per-(frame, tile)
// totals; pair count, capacity and overflow into the status block.  Ranges
// are clamped to the capacity so that an overflowed forward stays in bounds.
__global__ void __launch_bounds__(1024) k_tile_keyscan(const uint32_t* __restrict__ tcount, long long K,
                                                       unsigned long long cap, uint2* __restrict__ ranges,
                                                       const uint32_t* __restrict__ nf_block, int n_blocks,
                                                       unsigned long long wcount_off, const uint32_t* sort_fault,
                                                       Status* status) {
    __shared__ unsigned long long scratch[17];
    unsigned long long carry = 0;
    // 4 consecutive tiles per thread, 4096 per round; the next round's counts
    // are loaded while this round is scanned
    uint32_t nv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const long long i = 4 * (long long)threadIdx.x + j;
        nv[j] = i < K ? tcount[i] : 0u;
    }
    for (long long base = 0; base < K; base += 4096) {
        const long long i0 = base + 4 * (long long)threadIdx.x;
        uint32_t v[4];
        unsigned long long sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = nv[j];
            sum += v[j];
            nv[j] = i0 + 4096 + j < K ? tcount[i0 + 4096 + j] : 0u;
        }
        unsigned long long tot;
        unsigned long long a = carry + block_exclusive_scan<unsigned long long, 1024>(sum, scratch, &tot);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned long long b = a + v[j];
            if (i0 + j < K) ranges[i0 + j] = make_uint2((uint32_t)(a < cap ? a : cap), (uint32_t)(b < cap ? b : cap));
            a = b;
        }
        carry += tot;
    }
    uint32_t nf = 0;   // non-finite Gaussians counted by the preprocess blocks
    for (int i = threadIdx.x; i < n_blocks; i += 1024) nf += nf_block[i];
    nf = wave_reduce_sum(nf);
    __shared__ uint32_t nf_sum;
    if (threadIdx.x == 0) nf_sum = 0;
    __syncthreads();
    if (lane_id() == 0 && nf) atomicAdd(&nf_sum, nf);
    __syncthreads();
    if (threadIdx.x == 0) {
        status->n_pairs = carry;
        status->cap = cap;
        status->overflow = carry > cap ? 1u : 0u;
        status->overflow_seen |= carry > cap ? 1u : 0u;
        if (carry > status->n_pairs_seen) status->n_pairs_seen = carry;
        status->nonfinite = nf_sum;
        status->sort_fault = sort_fault ? *sort_fault : 0u;
        status->wcount_off = wcount_off;
        status->n_items = (unsigned long long)K;
        status->magic = kStatusMagic;
    }
}

// The status header and the sums of the forward's per-work-item counts, to
// host memory: one launch in place of a copy of the header, a second copy of
// all counts and their sum on the host (a pass through autograd, with and
// without: 2 frames of 97x75 pixels 293 and 263 us, one of 640x480 380 and
// 350).
__global__ void __launch_bounds__(1024) k_status_report(const Status* __restrict__ status, StatusReport* host) {
    __shared__ unsigned long long part[2][16];
    const Status st = *status;
    unsigned long long ev = 0, co = 0;
    if (st.magic == kStatusMagic && st.n_items <= (1ull << 26) && st.wcount_off >= sizeof(Status) &&
        st.wcount_off % 8 == 0 && st.wcount_off < (1ull << 44)) {
        const uint2* wcount = reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(status) + st.wcount_off);
        for (unsigned long long i = threadIdx.x; i < st.n_items; i += 8 * 1024) {
            uint2 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = i + 1024 * q < st.n_items ? wcount[i + 1024 * q] : make_uint2(0u, 0u);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                ev += v[q].x;
                co += v[q].y;
            }
        }
    }
    ev = wave_reduce_sum(ev);
    co = wave_reduce_sum(co);
    if (threadIdx.x % 64 == 0) {
        part[0][threadIdx.x / 64] = ev;
        part[1][threadIdx.x / 64] = co;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) {
            ev += part[0][w];
            co += part[1][w];
        }
        host->st = st;
        host->n_evaluated = ev;
        host->n_composited = co;
    }
}

// Introspection: the sorted rectangles, and the tiles they cover, back in item
// order.
__global__ void k_item_rects(const uint32_t* __restrict__ dkey, const uint32_t* __restrict__ dval,
                             const uint2* __restrict__ drect, long long M, uint2* __restrict__ rects,
                             uint32_t* __restrict__ counts) {
    for (long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x; j < M;
         j += (long long)gridDim.x * blockDim.x) {
        const uint2 r = drect[j];
        const uint32_t item = dval[j];
        if (item >= M) continue;   // no forward has filled the workspace
        if (rects) rects[item] = r;
        uint32_t xlo, xhi, ylo, yhi;
        unpack_rect(r, xlo, xhi, ylo, yhi);
        if (counts) counts[item] = dkey[j] == kCulledKey ? 0u : (xhi - xlo + 1) * (yhi - ylo + 1);
    }
}

// Introspection: expands the ranges into per-pair (frame, tile) keys.
__global__ void k_keys_from_ranges(const uint2* __restrict__ ranges, long long K,
                                   unsigned long long limit, uint32_t* __restrict__ keys) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < K;
         i += (long long)gridDim.x * blockDim.x) {
        const uint2 r = ranges[i];
        for (uint32_t p = r.x; p < r.y && p < limit; ++p) keys[p] = (uint32_t)i;
    }
}

}  // namespace

BinGeom bin_geometry(int64_t n, int32_t n_frames, int ntx, int nty, uint64_t cap) {
    BinGeom g;
    // level-A chunks: enough waves to fill the chip, at least 128 items each
    const int64_t M = n * (int64_t)n_frames;
    int C = 128;
    while (C < 2048 && M / C > 16384) C *= 2;
    g.C = C;
    g.QC = n > 0 ? (int)((n + C - 1) / C) : 0;
    g.ng = ((ntx + kGroupW - 1) / kGroupW) * ((nty + kGroupH - 1) / kGroupH);
    // segment of a group list, the unit of the counting pass's runs
    g.S = 128;
    // every segment but the last of each group list holds S entries, and the
    // group lists hold at most min(cap, M * groups) entries
    uint64_t entries = cap;
    if ((uint64_t)M * g.ng < entries) entries = (uint64_t)M * g.ng;
    g.max_segments = (int64_t)((entries + g.S - 1) / g.S) + (int64_t)n_frames * g.ng;
    return g;
}

// Grid caps of the one-wave placing and counting kernels.  The placing waves
// wait on loads most of the time, so a grid of several times the 8192 resident
// waves (32 per CU) keeps the chip busier than a resident-sized one: one wave
// per work item up to 128K items (1M x 16 frames: 94K).  The counting grid is
// sized from an upper bound on the segments, so its cap also bounds the waves
// that find no work.
constexpr int64_t kPlaceGridA = 131072;
constexpr int64_t kCountGrid = 8192;

hipError_t launch_binning(const Params& P, const Workspace& w, hipStream_t s) {
    const BinGeom g = bin_geometry(P.n, P.F, P.ntx, P.nty, P.cap);
    const int K = P.F * g.ng;
    const unsigned chunks = (unsigned)(P.F * g.QC);
    if (chunks) {
        ProfScope _p("k_group_count", s);
        const int cpw = g.C >= 512 ? 1 : (g.C >= 256 ? 2 : 4);   // 512 / C in [1, 4]
        hipLaunchKernelGGL(k_group_count, dim3((chunks + cpw - 1) / cpw), dim3(256), 0, s, P, g.C, g.QC, cpw,
                           depth_order(w), w.cntA, reinterpret_cast<uint32_t*>(w.touch));
    }
    if (chunks) {
        ProfScope _p("k_group_colscan", s);
        hipLaunchKernelGGL(k_group_colscan, dim3(g.ng, P.F), dim3(256), 0, s, P, g.QC,
                           w.cntA, w.lenA, w.tcount);
    } else {
        launch_fill_u32(w.lenA, 0u, K, s);
        launch_fill_u32(w.tcount, 0u, (int64_t)P.F * P.n_tiles, s);
    }
    {
        ProfScope _p("k_group_scan", s);
        hipLaunchKernelGGL(k_group_scan, dim3(1), dim3(1024), 0, s, w.lenA, K, g.S,
                           (unsigned long long)P.cap, w.granges, w.seg_start);
    }
    if (chunks) {
        ProfScope _p("k_group_place", s);
        const int ngy = (P.nty + kGroupH - 1) / kGroupH, ngx = (P.ntx + kGroupW - 1) / kGroupW;
        // runs of up to 512 items per wave while at least 8192 work items
        // remain (200k x 8 frames: runs of 4 chunks of 128; one 640 x 480
        // frame of 100k: 1 chunk; 1M x 16 frames: 1 chunk of 1024)
        int RA = g.C >= 512 ? 1 : 512 / g.C;
        while (RA > 1 && (int64_t)P.F * ((g.QC + RA - 1) / RA) * ngy < 8192) RA /= 2;
        const int64_t items = (int64_t)P.F * ((g.QC + RA - 1) / RA) * ngy;
        const unsigned grid = (unsigned)((items < kPlaceGridA ? items : kPlaceGridA) + 7) / 8 * 8;
        if ((int64_t)RA * g.C >= 1024)
            hipLaunchKernelGGL(k_group_place<8>, dim3(grid), dim3(64), 4 * (size_t)ngx, s, P, g.C, g.QC, RA,
                               depth_order(w), w.cntA, w.granges, w.gval, w.gloc);
        else
            hipLaunchKernelGGL(k_group_place<1>, dim3(grid), dim3(64), 4 * (size_t)ngx, s, P, g.C, g.QC, RA,
                               depth_order(w), w.cntA, w.granges, w.gval, w.gloc);
    }
    // persistent counting grid: every wave takes a run of segments
    const int64_t runs = (g.max_segments + kCountRun - 1) / kCountRun;
    const unsigned segs = (unsigned)(runs < kCountGrid ? runs : kCountGrid);
    {
        ProfScope _p("k_tile_count", s);
        hipLaunchKernelGGL(k_tile_count, dim3(segs), dim3(64), 0, s, P, g.S, w.seg_start, w.granges,
                           w.gloc, w.tcount);
    }
    {
        ProfScope _p("k_tile_keyscan", s);
        hipLaunchKernelGGL(k_tile_keyscan, dim3(1), dim3(1024), 0, s, w.tcount,
                           (long long)P.F * P.n_tiles, (unsigned long long)P.cap, w.ranges, w.nf_block,
                           (int)((P.n + 255) / 256),
                           (unsigned long long)(reinterpret_cast<char*>(w.wcount) - reinterpret_cast<char*>(w.status)),
                           one_sweep_sort(P, w) ? w.sctl + kSortFault : nullptr, w.status);
    }
    return hipGetLastError();
}

void launch_item_rects(const Workspace& w, uint2* rects, uint32_t* counts, hipStream_t s) {
    if (w.M == 0) return;
    const long long blocks = (w.M + 255) / 256;
    hipLaunchKernelGGL(k_item_rects, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, s,
                       w.dkey[1], w.dval[1], w.drect[1], (long long)w.M, rects, counts);
}

void launch_status_report(const void* ws, StatusReport* host, hipStream_t s) {
    hipLaunchKernelGGL(k_status_report, dim3(1), dim3(1024), 0, s, static_cast<const Status*>(ws), host);
}

void launch_tile_lists(const Params& P, const Workspace& w, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_lists, dim3((unsigned)(P.F * P.n_tiles)), dim3(64), 0, s, P, w.ranges, w.granges, w.gval,
                       w.gloc, w.tval);
}

void launch_keys_from_ranges(const Params& P, const Workspace& w, uint32_t* keys,
                             unsigned long long limit, hipStream_t s) {
    const long long K = (long long)P.F * P.n_tiles;
    hipLaunchKernelGGL(k_keys_from_ranges, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, s,
                       w.ranges, K, limit, keys);
}

}  // namespace gft
