// Tile lists read straight from the group lists (shared by bin.hip, which
// builds the group lists, and composite.hip, which walks them).
//
// A group list holds the items that touch one group of 8x8 tiles, in depth
// order, each with its tile rectangle clipped to the group (16 bits).  The
// list of one tile is the subsequence of entries whose rectangle holds the
// tile, so a wave that needs a tile's list filters its group's.
#pragma once

#include "common.h"

namespace gft {

constexpr int kGroupW = 8, kGroupH = 8;   // tiles per group

// A clipped rectangle [x0, x1] x [y0, y1] in group coordinates (0..7), packed
// as the four values x0, 7 - x1, y0, 7 - y1 with a clear bit above each.  It
// holds tile (x, y) iff none of them exceeds that of the one-tile rectangle
// (x, x, y, y): with the clear bits set in the latter, a subtraction leaves
// all four set exactly then, for two packed rectangles of a word at once.
__host__ __device__ constexpr uint32_t pack_rect(uint32_t x0, uint32_t x1, uint32_t y0, uint32_t y1) {
    return x0 | ((7u - x1) << 4) | (y0 << 8) | ((7u - y1) << 12);
}
constexpr uint32_t kRectGuards = 0x8888u;
constexpr uint32_t kEmptyRect = pack_rect(7, 0, 7, 0);   // holds no tile

struct LocalRect {
    uint32_t x0, x1, y0, y1;
};

__device__ __forceinline__ LocalRect local_rect(uint32_t packed) {
    LocalRect r;
    r.x0 = packed & 7u;
    r.x1 = 7u - ((packed >> 4) & 7u);
    r.y0 = (packed >> 8) & 7u;
    r.y1 = 7u - ((packed >> 12) & 7u);
    return r;
}

// Lane masks held in scalar registers: the lanes whose condition (one
// comparison, which then writes the mask itself) is true, and back.
__device__ __forceinline__ uint64_t lanes(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ bool lane_of(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// Lanes of `peers` below this one, plus `more`.
__device__ __forceinline__ uint32_t rank_below(uint64_t peers, uint32_t more = 0u) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, more));
}

// The walk over a group list for one tile by NW waves, 256 entries a round and
// wave (four consecutive ones per lane, one 8-byte load); the next round's are
// in flight while the caller works on those it has.
template <int NW>
struct TileWalk {
    const uint16_t* gloc;
    uint32_t beg, at, end;   // entries of the group list; `at` the round loaded (wave 0's part)
    uint32_t mine;           // this lane's first entry of the round, from `at`
    uint32_t tile;           // the tile's packed rectangle with guards, twice
    uint2 word;

    // the lanes whose first .. fourth entry of a round holds the tile
    struct Hits {
        uint64_t m0, m1, m2, m3;
        uint32_t entry;
        __device__ __forceinline__ uint32_t count() const {
            return (uint32_t)(__popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3));
        }
        // hands this lane's to put(entry index, position among the wave's)
        template <typename Put>
        __device__ __forceinline__ void each(Put put) const {
            if ((m0 | m1 | m2 | m3) == 0ull) return;
            uint32_t pos = rank_below(m0, rank_below(m1, rank_below(m2, rank_below(m3))));
            if (lane_of(m0)) put(entry, pos++);
            if (lane_of(m1)) put(entry + 1u, pos++);
            if (lane_of(m2)) put(entry + 2u, pos++);
            if (lane_of(m3)) put(entry + 3u, pos);
        }
    };

    __device__ __forceinline__ void load() {
        const uint32_t j = at + mine;   // a multiple of 4: 8-byte aligned
        word = make_uint2(kEmptyRect * 0x10001u, kEmptyRect * 0x10001u);
        if (j < end) {
            word = *reinterpret_cast<const uint2*>(gloc + j);
            if (j < beg || j + 4u > end) {   // the list starts or ends inside the word
                if (j < beg) word.x = (word.x & 0xffff0000u) | kEmptyRect;
                if (j + 1u < beg || j + 1u >= end) word.x = (word.x & 0xffffu) | (kEmptyRect << 16);
                if (j + 2u < beg || j + 2u >= end) word.y = (word.y & 0xffff0000u) | kEmptyRect;
                if (j + 3u >= end) word.y = (word.y & 0xffffu) | (kEmptyRect << 16);
            }
        }
    }

    __device__ __forceinline__ bool more() const { return at < end; }

    // The round's hits; the next round's load is issued.
    __device__ __forceinline__ Hits round() {
        const uint32_t g = kRectGuards * 0x10001u;
        const uint32_t a = (tile - word.x) & g, b = (tile - word.y) & g;
        Hits h;
        h.m0 = lanes((uint16_t)a == (uint16_t)kRectGuards);
        h.m1 = lanes(a >= (kRectGuards << 16));
        h.m2 = lanes((uint16_t)b == (uint16_t)kRectGuards);
        h.m3 = lanes(b >= (kRectGuards << 16));
        h.entry = at + mine;
        at += 256u * NW;
        load();
        return h;
    }
};

// The walk of tile (tx, ty) of frame f, its first round in flight.
template <int NW>
__device__ __forceinline__ TileWalk<NW> tile_walk(const Params& P, int f, int tx, int ty,
                                                  const uint2* __restrict__ granges,
                                                  const uint16_t* __restrict__ gloc, int wave, int lane) {
    const int ngx = (P.ntx + kGroupW - 1) / kGroupW, ngy = (P.nty + kGroupH - 1) / kGroupH;
    const uint2 gr = granges[((size_t)f * ngy + ty / kGroupH) * ngx + tx / kGroupW];
    const uint32_t x = (uint32_t)tx % kGroupW, y = (uint32_t)ty % kGroupH;
    TileWalk<NW> g;
    g.gloc = gloc;
    g.beg = gr.x;
    g.at = gr.x & ~3u;
    g.end = gr.y;
    g.mine = 256u * (uint32_t)wave + 4u * (uint32_t)lane;
    g.tile = (pack_rect(x, x, y, y) | kRectGuards) * 0x10001u;
    g.load();
    return g;
}

}  // namespace gft
