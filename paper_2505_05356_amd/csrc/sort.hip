// Depth ordering of the (frame, Gaussian) items.
//
// Every pixel composites the Gaussians of its tile front to back (paper §3),
// in ascending (depth key, Gaussian index) order per frame.  The M = F * N
// items start in (frame, index) order; a stable LSD radix sort over their
// 32-bit depth keys, run segment by segment (one segment per frame), leaves
// them frame-major and depth-ordered inside each frame, ties in index order.
// The tile lists are then built from this order by the binning kernels
// (bin.hip) without sorting any (tile, Gaussian) pairs.
//
// Digits are taken from the key minus the bits of near_z, below which no item
// is valid: 27 bits then hold 16 octaves of depth (0.2 m to 13 km), so three
// passes of 9 bits sort them.  A fourth pass over the upper 5 bits is launched
// every time and returns at once unless some valid key needs it (sctl[
// kSortWide], which also tells the readers the buffer that holds the result).
// Each pass moves every item once and waits on its launches; four passes of 8
// bits took a third more of both (whole sort of 16 frames of 1M items: 745 us
// then, 543 now; a forward pass over one frame of 100k: 115 us then, 107 now).
//
// Radix passes are reduce-then-scan (upsweep tile histograms, column scan per
// (frame, digit), downsweep rank-and-scatter) with no inter-workgroup
// waiting.  Batches of few sort tiles, where those three launches per pass
// cost more than the work, instead count the digits of all passes in one
// launch and sort each pass in one launch: a workgroup takes the next
// sort tile from an atomic counter, ranks its keys, publishes its per-digit
// counts and adds those of the frame's earlier tiles by decoupled look-back
// (a bounded wait: those tiles were taken earlier, so their workgroups are
// running), then scatters.  Small frames are each sorted by one workgroup in
// LDS.  Sort tiles never straddle a frame.  Each item's
// tile rectangle rides along as payload, so the binning kernels read it in
// depth order without gathering it by item id; the item id itself is first
// written by the first pass (it is the position there).  Ranking inside a
// tile is stable: wave-level peer matching with ballots, wave-private digit
// counters in LDS, then an LDS reorder so that each digit run is written
// contiguously.
#include <cstring>

#include "block_scan.h"
#include "common.h"

namespace gft {

namespace {

// Sort tile `g` of the segmented layout (TILE keys): frame and element range.
struct SortTile {
    long long f, t, beg, end;
};

template <int TILE>
__device__ __forceinline__ SortTile sort_tile(long long g, long long n, long long tpf) {
    SortTile r;
    r.f = g / tpf;
    r.t = g - r.f * tpf;
    r.beg = r.f * n + r.t * TILE;
    r.end = min(r.beg + TILE, (r.f + 1) * n);
    return r;
}

// The digits' source: monotonic in the key for valid keys (no valid key is
// below `base`), all ones for a culled one.
__device__ __forceinline__ uint32_t key_digits(uint32_t key, uint32_t base) {
    return key == kCulledKey ? key : key - base;
}
__device__ __forceinline__ bool key_wide(uint32_t key, uint32_t base) {
    return key != kCulledKey && key - base >= (1u << kSortWideShift) - 1u;
}

// Those of the lanes `among` whose low BITS bits of d equal this lane's: per
// bit, the lanes that have it, complemented where this lane has not.
template <int BITS>
__device__ __forceinline__ uint64_t peers_of(uint32_t d, uint64_t among) {
    uint32_t lo = (uint32_t)among, hi = (uint32_t)(among >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const int32_t m = (int32_t)(d << (31 - b)) >> 31;   // -1 where the bit is set
        const uint64_t set = __builtin_amdgcn_ballot_w64(m < 0);
        lo &= ~((uint32_t)set ^ (uint32_t)m);
        hi &= ~((uint32_t)(set >> 32) ^ (uint32_t)m);
    }
    return (uint64_t)hi << 32 | lo;
}

// One pass of a sort tile of NT threads, 8 keys each.  Bound by the time that
// the items of one tile spend waiting between barriers, so by the workgroups
// that share a CU: the payload goes through the same LDS after the keys (35 KB
// per tile of 4096 items in place of 68) and is loaded only after the ranking
// (80 registers in place of 133).  Downsweep of 16M items per pass: 146 us
// (3.5 TB/s of its 512 MB) against 179 with all of a tile's items in LDS and
// registers at once.
template <int NT>
struct TileSort {
    static constexpr int TILE = NT * kSortItems, WAVES = NT / 64, DPT = kSortBuckets / NT;
    static_assert(DPT >= 1 && WAVES * kSortBuckets <= TILE, "digit counters share the keys' LDS");
    struct Shared {
        // the waves' digit counters [WAVES][kSortBuckets], then the sorted
        // (key, item) pairs, then the sorted rectangles: one after the other,
        // so that several workgroups share a CU
        uint2 pair[TILE];
        uint32_t out_base[kSortBuckets];
        uint32_t scratch[16];
    };
    uint32_t k[kSortItems], v[kSortItems], rank[kSortItems];
    uint2 rc[kSortItems];

    __device__ static uint32_t* counters(Shared& S) { return reinterpret_cast<uint32_t*>(S.pair); }

    __device__ __forceinline__ void clear(Shared& S, int wave, int lane) {
#pragma unroll
        for (int i = 0; i < kSortBuckets / 64; ++i) counters(S)[wave * kSortBuckets + i * 64 + lane] = 0u;
    }

    // keys of this tile; at: tid's first element
    __device__ __forceinline__ void load_keys(const SortTile& st, uint32_t at, uint32_t valid,
                                              const uint32_t* __restrict__ kin) {
        const uint32_t* kt = kin + st.beg;
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) k[it] = at + 64 * it < valid ? kt[at + 64 * it] : 0u;
    }

    // Issued once the keys are ranked (the ranking needs the registers), to
    // arrive while the digits are scanned.  vin NULL: the items are still in
    // item order.
    __device__ __forceinline__ void load_payload(const SortTile& st, uint32_t at, uint32_t valid,
                                                 const uint32_t* __restrict__ vin, const uint2* __restrict__ rin) {
        const uint32_t* vt = vin + st.beg;
        const uint2* rt = rin + st.beg;
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            v[it] = vin ? (at + 64 * it < valid ? vt[at + 64 * it] : 0u) : (uint32_t)st.beg + at + 64 * it;
            rc[it] = at + 64 * it < valid ? rt[at + 64 * it] : make_uint2(0u, 0u);
        }
    }

    // rank[it]: the key's rank among its wave's keys of the same digit
    __device__ __forceinline__ void rank_in_wave(Shared& S, uint32_t at, uint32_t valid_n, int wave, int shift,
                                                 uint32_t base) {
        // Wave-synchronous LDS counter: every lane of the peer group reads
        // the counter, then its highest lane advances it.  LDS operations
        // of one wave complete in issue order and the volatile accesses
        // keep the compiler from reordering them across iterations; the
        // pointer keeps its LDS address space, so they stay LDS
        // instructions rather than generic (flat) ones.
        volatile __attribute__((address_space(3))) uint32_t* wh =
            (volatile __attribute__((address_space(3))) uint32_t*)(counters(S) + wave * kSortBuckets);
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            const bool valid = at + 64 * it < valid_n;
            const uint32_t d = key_digits(k[it], base) >> shift & (kSortBuckets - 1);
            const uint64_t peers = peers_of<kDigitBits>(d, __builtin_amdgcn_ballot_w64(valid));
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            const uint32_t cnt = (uint32_t)__popcll(peers);
            uint32_t prev = 0;
            if (valid) prev = wh[d];
            if (valid && below == cnt - 1) wh[d] = prev + cnt;
            rank[it] = prev + below;
            // one key's peers at a time: all eight at once take twice the registers
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // After every wave has ranked: the tile's count of this thread's digits
    // (digit tid * DPT + e), and the counters replaced by the position of the
    // wave's first key of the digit within the sorted tile; start: the
    // position of the digit.
    __device__ __forceinline__ void digit_starts(Shared& S, int tid, uint32_t (&count)[DPT], uint32_t (&start)[DPT]) {
        uint32_t c[DPT][WAVES], all = 0;
#pragma unroll
        for (int e = 0; e < DPT; ++e) {
            count[e] = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                c[e][w] = counters(S)[w * kSortBuckets + tid * DPT + e];
                count[e] += c[e][w];
            }
            all += count[e];
        }
        uint32_t tot;
        uint32_t run = block_exclusive_scan<uint32_t, NT>(all, S.scratch, &tot);
#pragma unroll
        for (int e = 0; e < DPT; ++e) {
            start[e] = run;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                counters(S)[w * kSortBuckets + tid * DPT + e] = run;
                run += c[e][w];
            }
        }
    }

    // Exclusive scan over all digits of one value per digit.
    __device__ static __forceinline__ void scan_digits(Shared& S, const uint32_t (&val)[DPT], uint32_t (&out)[DPT]) {
        uint32_t all = 0, tot;
#pragma unroll
        for (int e = 0; e < DPT; ++e) all += val[e];
        uint32_t run = block_exclusive_scan<uint32_t, NT>(all, S.scratch, &tot);
#pragma unroll
        for (int e = 0; e < DPT; ++e) {
            out[e] = run;
            run += val[e];
        }
    }

    // S.out_base[d]: output position of the tile's sorted element j of digit
    // d, minus j (mod 2^32: the true position is below n).  Starts with a
    // barrier and leaves the tile's LDS in use.
    __device__ __forceinline__ void scatter(Shared& S, const SortTile& st, uint32_t at, uint32_t valid, int wave,
                                            int shift, uint32_t base, long long n, uint32_t* __restrict__ kout,
                                            uint32_t* __restrict__ vout, uint2* __restrict__ rout) {
        const uint32_t tid = threadIdx.x;
        kout += st.f * n;
        vout += st.f * n;
        rout += st.f * n;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kSortItems; ++it)
            rank[it] += counters(S)[wave * kSortBuckets + (key_digits(k[it], base) >> shift & (kSortBuckets - 1))];
        __syncthreads();   // the counters' LDS becomes the pairs'
#pragma unroll
        for (int it = 0; it < kSortItems; ++it)
            if (at + 64 * it < valid) S.pair[rank[it]] = make_uint2(k[it], v[it]);
        __syncthreads();
        uint32_t to[kSortItems];   // output position in the frame
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            const uint32_t j = tid + it * NT;
            if (j < valid) {
                const uint2 p = S.pair[j];
                to[it] = S.out_base[key_digits(p.x, base) >> shift & (kSortBuckets - 1)] + j;
                kout[to[it]] = p.x;
                vout[to[it]] = p.y;
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kSortItems; ++it)
            if (at + 64 * it < valid) S.pair[rank[it]] = rc[it];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            const uint32_t j = tid + it * NT;
            if (j < valid) rout[to[it]] = S.pair[j];
        }
    }
};

// counts[(f * tpf + t) * kSortBuckets + d] = keys of digit d in tile t of
// frame f.  CP copies of each wave's histogram, lane l counting into copy
// l % CP: the third digit of depths takes few values, so its counts would
// otherwise serialise on a few LDS addresses.  Pass 0 also finds out whether
// the fourth pass is needed.
template <int CP>
__global__ void __launch_bounds__(kBigThreads) k_sort_upsweep(const uint32_t* __restrict__ keys, long long n, int F,
                                                              long long tpf, int pass, uint32_t base,
                                                              uint32_t* __restrict__ counts,
                                                              uint32_t* __restrict__ sctl) {
    constexpr int TILE = TileSort<kBigThreads>::TILE, WAVES = kBigThreads / 64;
    __shared__ uint32_t hist[WAVES * CP][kSortBuckets];
    if (pass == kSortPasses && sctl[kSortWide] == 0u) return;
    const int shift = kDigitBits * pass;
    const int copy = (threadIdx.x / 64) * CP + (int)(threadIdx.x % CP);
    const long long ntiles = (long long)F * tpf;
    for (long long g = blockIdx.x; g < ntiles; g += gridDim.x) {
        const SortTile st = sort_tile<TILE>(g, n, tpf);
        for (int i = threadIdx.x; i < WAVES * CP * kSortBuckets; i += kBigThreads) (&hist[0][0])[i] = 0;
        // a histogram needs no element order: each thread loads its 8 keys
        // as two 16-byte vectors where the tile is whole and 16-byte aligned,
        // all loads in flight before the first count
        uint32_t kv[kSortItems];
        const long long i0 = st.beg + (long long)threadIdx.x * 4;
        const bool vec = st.end - st.beg == TILE && (st.beg & 3) == 0;
        if (vec) {
            const uint4 a = *reinterpret_cast<const uint4*>(keys + i0);
            const uint4 b = *reinterpret_cast<const uint4*>(keys + i0 + 4 * kBigThreads);
            kv[0] = a.x, kv[1] = a.y, kv[2] = a.z, kv[3] = a.w;
            kv[4] = b.x, kv[5] = b.y, kv[6] = b.z, kv[7] = b.w;
        } else {
#pragma unroll
            for (int it = 0; it < kSortItems; ++it) {
                const long long idx = st.beg + it * kBigThreads + threadIdx.x;
                kv[it] = idx < st.end ? keys[idx] : kCulledKey;
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            const bool ok = vec || st.beg + it * kBigThreads + threadIdx.x < st.end;
            if (ok) atomicAdd(&hist[copy][key_digits(kv[it], base) >> shift & (kSortBuckets - 1)], 1u);
        }
        if (pass == 0) {
            bool wide = false;
#pragma unroll
            for (int it = 0; it < kSortItems; ++it) wide |= key_wide(kv[it], base);
            if (wide) sctl[kSortWide] = 1u;
        }
        __syncthreads();
        for (int d = threadIdx.x; d < kSortBuckets; d += kBigThreads) {
            uint32_t c = 0;
#pragma unroll
            for (int q = 0; q < WAVES * CP; ++q) c += hist[q][d];
            counts[g * kSortBuckets + d] = c;
        }
        __syncthreads();
    }
}

// grid (kSortBuckets / 32, F): exclusive scan over the frame's tiles of the
// counts of 32 digits (a 128-byte run of every tile's row), each of 32 groups
// of threads a run of consecutive tiles; the totals go to
// totals[f * kSortBuckets + d].
constexpr int kScanDigits = 32, kScanRuns = 32;
__global__ void __launch_bounds__(kScanDigits* kScanRuns) k_sort_scan(uint32_t* __restrict__ counts, int tpf, int pass,
                                                                      uint32_t* __restrict__ totals,
                                                                      const uint32_t* __restrict__ sctl) {
    __shared__ uint32_t sums[kScanRuns][kScanDigits];
    if (pass == kSortPasses && sctl[kSortWide] == 0u) return;
    const int dl = threadIdx.x % kScanDigits, run = threadIdx.x / kScanDigits;
    const int d = blockIdx.x * kScanDigits + dl, f = blockIdx.y;
    const int per = (tpf + kScanRuns - 1) / kScanRuns;
    const int t0 = min(run * per, tpf), t1 = min(t0 + per, tpf);
    uint32_t* col = counts + (size_t)f * tpf * kSortBuckets + d;
    uint32_t s = 0;
    for (int t = t0; t < t1; t += 8) {
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = t + i < t1 ? col[(size_t)(t + i) * kSortBuckets] : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) s += v[i];
    }
    sums[run][dl] = s;
    __syncthreads();
    uint32_t at = 0, total = 0;
#pragma unroll
    for (int r = 0; r < kScanRuns; ++r) {
        const uint32_t c = sums[r][dl];
        at += r < run ? c : 0u;
        total += c;
    }
    for (int t = t0; t < t1; t += 8) {
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = t + i < t1 ? col[(size_t)(t + i) * kSortBuckets] : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (t + i < t1) col[(size_t)(t + i) * kSortBuckets] = at;
            at += v[i];
        }
    }
    if (run == 0) totals[f * kSortBuckets + d] = total;
}

__global__ void __launch_bounds__(kBigThreads) k_sort_downsweep(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, const uint2* __restrict__ rin,
    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, uint2* __restrict__ rout, long long n,
    long long tpf, int pass, uint32_t base, const uint32_t* __restrict__ counts,
    const uint32_t* __restrict__ totals, const uint32_t* __restrict__ sctl) {
    using Sort = TileSort<kBigThreads>;
    __shared__ Sort::Shared S;
    if (pass == kSortPasses && sctl[kSortWide] == 0u) return;
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, shift = kDigitBits * pass;
    // consecutive tiles write adjacent runs of every digit: one XCD.  One tile
    // per workgroup: under a loop over tiles the compiler kept some 60
    // loop-invariant addresses in registers.
    const long long g = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const SortTile st = sort_tile<Sort::TILE>(g, n, tpf);
    const uint32_t at = wave * (kSortItems * 64) + lane, valid = (uint32_t)(st.end - st.beg);
    Sort T;
    T.load_keys(st, at, valid, kin);
    // this tile's offset of the thread's digits among the frame's keys of the
    // digit, and the frame's counts, loaded now to overlap the ranking
    uint32_t off[Sort::DPT], fcount[Sort::DPT], fbase[Sort::DPT];
#pragma unroll
    for (int e = 0; e < Sort::DPT; ++e) {
        off[e] = counts[g * kSortBuckets + tid * Sort::DPT + e];
        fcount[e] = totals[st.f * kSortBuckets + tid * Sort::DPT + e];
    }
    T.clear(S, wave, lane);
    T.rank_in_wave(S, at, valid, wave, shift, base);
    T.load_payload(st, at, valid, vin, rin);
    __syncthreads();
    uint32_t count[Sort::DPT], start[Sort::DPT];
    T.digit_starts(S, tid, count, start);
    Sort::scan_digits(S, fcount, fbase);
#pragma unroll
    for (int e = 0; e < Sort::DPT; ++e) S.out_base[tid * Sort::DPT + e] = fbase[e] + off[e] - start[e];
    T.scatter(S, st, at, valid, wave, shift, base, n, kout, vout, rout);
}

// Digit counts of every pass of the one-sweep sort: shist[(f * (kSortPasses +
// 1) + pass) * kSortBuckets + d] += keys of frame f whose digit `pass` is d
// (the key multiset is the same in every pass).  One workgroup per sort tile,
// which also clears the tile's look-back words of the first pass and finds
// out whether the fourth pass is needed.
__global__ void __launch_bounds__(kSortThreads) k_sort_hist(const uint32_t* __restrict__ keys, long long n,
                                                            long long tpf, uint32_t base,
                                                            uint32_t* __restrict__ shist,
                                                            uint32_t* __restrict__ look0,
                                                            uint32_t* __restrict__ sctl) {
    constexpr int TILE = TileSort<kSortThreads>::TILE, WAVES = kSortThreads / 64;
    __shared__ uint32_t hist[WAVES][kSortPasses][kSortBuckets];
    __shared__ uint32_t top[1 << (32 - kSortWideShift)];
    const long long g = blockIdx.x;
    const SortTile st = sort_tile<TILE>(g, n, tpf);
    const int tid = threadIdx.x, wave = tid / 64;
    uint32_t kv[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const long long idx = st.beg + it * kSortThreads + tid;
        kv[it] = idx < st.end ? keys[idx] : kCulledKey;
    }
    for (int d = tid; d < kSortBuckets; d += kSortThreads) look0[g * kSortBuckets + d] = 0u;
    for (int i = tid; i < WAVES * kSortPasses * kSortBuckets; i += kSortThreads) (&hist[0][0][0])[i] = 0u;
    if (tid < (1 << (32 - kSortWideShift))) top[tid] = 0u;
    __syncthreads();
    bool wide = false;
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        if (st.beg + it * kSortThreads + tid < st.end) {
            const uint32_t r = key_digits(kv[it], base);
#pragma unroll
            for (int p = 0; p < kSortPasses; ++p)
                atomicAdd(&hist[wave][p][r >> (kDigitBits * p) & (kSortBuckets - 1)], 1u);
            // nearly every key's upper bits are 0: those are counted as the rest
            if (r >> kSortWideShift) atomicAdd(&top[r >> kSortWideShift], 1u);
            wide |= key_wide(kv[it], base);
        }
    }
    if (wide) sctl[kSortWide] = 1u;
    __syncthreads();
    uint32_t* out = shist + st.f * (kSortPasses + 1) * kSortBuckets;
#pragma unroll
    for (int p = 0; p < kSortPasses; ++p)
        for (int d = tid; d < kSortBuckets; d += kSortThreads) {
            uint32_t v = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) v += hist[w][p][d];
            if (v) atomicAdd(&out[p * kSortBuckets + d], v);
        }
    if (tid < (1 << (32 - kSortWideShift))) {
        uint32_t v = top[tid];
        if (tid == 0) {
            v = (uint32_t)(st.end - st.beg);
            for (int i = 1; i < (1 << (32 - kSortWideShift)); ++i) v -= top[i];
        }
        if (v) atomicAdd(&out[kSortPasses * kSortBuckets + tid], v);
    }
}

// Look-back word of (tile, pair of digits): per digit count << 2 | state in 32
// bits, state 1 = the tile's own counts, 2 = the inclusive counts of the
// frame's tiles up to this one.  Both digits are published in one store.
constexpr uint32_t kLookAggregate = 1u, kLookInclusive = 2u;
// A tile waits at most this many polls for an earlier tile to publish; past
// it the sort raises the fault flag (reported by gftorf_read_status) instead
// of waiting on.
constexpr int kLookSpinLimit = 1 << 22;
constexpr int kLookWindow = 16;   // earlier tiles a look-back reads at a time

__device__ __forceinline__ uint64_t look_load(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void look_store(uint64_t* p, uint32_t c0, uint32_t c1, uint32_t state) {
    __hip_atomic_store(p, (uint64_t)(c1 << 2 | state) << 32 | (c0 << 2 | state), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// One stable pass over digit `pass` of every frame's segment, one workgroup
// per sort tile.  look holds the pass's look-back words (cleared by the
// previous launch); look_next, if not NULL, is cleared here for the next pass.
__global__ void __launch_bounds__(kSortThreads) k_sort_onesweep(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, const uint2* __restrict__ rin,
    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, uint2* __restrict__ rout, long long n,
    long long tpf, int pass, uint32_t base, const uint32_t* __restrict__ shist, uint32_t* __restrict__ sctl,
    uint32_t* __restrict__ look, uint32_t* __restrict__ look_next) {
    using Sort = TileSort<kSortThreads>;
    __shared__ Sort::Shared S;
    __shared__ uint32_t s_tile;
    if (pass == kSortPasses && sctl[kSortWide] == 0u) return;

    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, shift = kDigitBits * pass;
    Sort T;
    // tiles are numbered in the order their workgroups start, so every tile
    // a workgroup waits for belongs to a workgroup that is already running
    if (tid == 0) s_tile = atomicAdd(&sctl[pass], 1u);
    T.clear(S, wave, lane);
    __syncthreads();
    const long long g = __builtin_amdgcn_readfirstlane((int)s_tile);
    const SortTile st = sort_tile<Sort::TILE>(g, n, tpf);
    const uint32_t at = wave * (kSortItems * 64) + lane, valid = (uint32_t)(st.end - st.beg);
    T.load_keys(st, at, valid, kin);
    uint32_t fcount[Sort::DPT];
#pragma unroll
    for (int e = 0; e < Sort::DPT; ++e) {
        if (look_next) look_next[g * kSortBuckets + tid * Sort::DPT + e] = 0u;
        fcount[e] = shist[(st.f * (kSortPasses + 1) + pass) * kSortBuckets + tid * Sort::DPT + e];
    }
    T.rank_in_wave(S, at, valid, wave, shift, base);
    T.load_payload(st, at, valid, vin, rin);
    __syncthreads();
    uint32_t count[Sort::DPT], start[Sort::DPT], fbase[Sort::DPT];
    T.digit_starts(S, tid, count, start);
    // the tile's place among the frame's tiles by look-back
    static_assert(Sort::DPT == 2, "a look-back word holds two digits");
    uint64_t* words = reinterpret_cast<uint64_t*>(look) + tid;   // of tile 0; kSortThreads per tile
    look_store(words + g * kSortThreads, count[0], count[1], st.t == 0 ? kLookInclusive : kLookAggregate);
    Sort::scan_digits(S, fcount, fbase);
    const long long first = st.f * tpf;
    uint32_t excl0 = 0, excl1 = 0;
    int spins = 0;
    for (long long j = g - 1; j >= first;) {
        // a window of earlier tiles per round trip (their words come from
        // beyond L2, about a microsecond each time)
        uint64_t wv[kLookWindow];
#pragma unroll
        for (int q = 0; q < kLookWindow; ++q)
            wv[q] = j - q >= first ? look_load(words + (j - q) * kSortThreads) : (uint64_t)kLookInclusive;
        int seen = 0;
        bool done = false;
#pragma unroll
        for (int q = 0; q < kLookWindow; ++q) {
            const uint32_t state = (uint32_t)wv[q] & 3u;
            if (done || seen < q || state == 0u) continue;
            excl0 += (uint32_t)wv[q] >> 2;
            excl1 += (uint32_t)(wv[q] >> 34);
            seen = q + 1;
            done = state == kLookInclusive;
        }
        j -= seen;
        if (done) break;
        if (seen == 0) {
            if (++spins > kLookSpinLimit) {
                sctl[kSortFault] = 1u;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    if (st.t != 0) look_store(words + g * kSortThreads, excl0 + count[0], excl1 + count[1], kLookInclusive);
    S.out_base[2 * tid] = fbase[0] + excl0 - start[0];
    S.out_base[2 * tid + 1] = fbase[1] + excl1 - start[1];
    T.scatter(S, st, at, valid, wave, shift, base, n, kout, vout, rout);
}

// Frames of at most kFrameSortMax items: one workgroup sorts a frame in LDS,
// all passes in one launch, and writes the result to buffer 1.  IT keys per
// thread.  Bound by its chain of barriers and LDS round trips, which is still
// shorter than that of five launches up to kFrameSortMax items.
constexpr int kFrameThreads = 1024;
template <int IT>
__global__ void __launch_bounds__(kFrameThreads) k_sort_frame(const uint32_t* __restrict__ kin,
                                                              const uint2* __restrict__ rin, uint32_t n, uint32_t base,
                                                              uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                              uint2* __restrict__ rout) {
    constexpr int WAVES = kFrameThreads / 64;
    static_assert(IT * kFrameThreads <= 65536, "positions in 16 bits");
    __shared__ uint2 pair[IT * kFrameThreads];
    __shared__ uint16_t cnt[WAVES][kSortBuckets];
    __shared__ uint32_t scratch[WAVES];
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const size_t first = (size_t)blockIdx.x * n;
    const uint32_t at = wave * (64 * IT) + lane;
    uint32_t k[IT], v[IT], rank[IT];
    bool wide = false;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        v[it] = at + 64 * it;
        k[it] = v[it] < n ? kin[first + v[it]] : kCulledKey;
        wide |= key_wide(k[it], base);
    }
    const int passes = __syncthreads_or(wide) ? kSortPasses + 1 : kSortPasses;
    volatile __attribute__((address_space(3))) uint16_t* wc =
        (volatile __attribute__((address_space(3))) uint16_t*)cnt[wave];
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = kDigitBits * pass;
        for (int i = lane; i < kSortBuckets / 2; i += 64) reinterpret_cast<uint32_t*>(cnt[wave])[i] = 0u;
#pragma unroll
        for (int it = 0; it < IT; ++it) {   // the ranking of TileSort
            const bool valid = at + 64 * it < n;
            const uint32_t d = key_digits(k[it], base) >> shift & (kSortBuckets - 1);
            const uint64_t peers = peers_of<kDigitBits>(d, __builtin_amdgcn_ballot_w64(valid));
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            const uint32_t c = (uint32_t)__popcll(peers);
            uint32_t prev = 0;
            if (valid) prev = wc[d];
            if (valid && below == c - 1) wc[d] = (uint16_t)(prev + c);
            rank[it] = prev + below;
        }
        __syncthreads();
        uint32_t c[WAVES], all = 0, tot;
        if (tid < kSortBuckets)
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                c[w] = cnt[w][tid];
                all += c[w];
            }
        uint32_t run = block_exclusive_scan<uint32_t, kFrameThreads>(all, scratch, &tot);
        if (tid < kSortBuckets)
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                cnt[w][tid] = (uint16_t)run;
                run += c[w];
            }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const uint32_t d = key_digits(k[it], base) >> shift & (kSortBuckets - 1);
            if (at + 64 * it < n) pair[wc[d] + rank[it]] = make_uint2(k[it], v[it]);
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const uint2 p = pair[at + 64 * it];   // past n: never written, never used
            k[it] = p.x;
            v[it] = p.y;
        }
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const uint32_t j = at + 64 * it;
        if (j < n) {
            kout[first + j] = k[it];
            vout[first + j] = (uint32_t)first + v[it];
            rout[first + j] = rin[first + v[it]];
        }
    }
}

// Introspection: a result that the fourth pass left in buffer 0, to buffer 1.
__global__ void k_sort_settle(const uint32_t* __restrict__ sctl, long long M, const uint32_t* __restrict__ k0,
                              const uint32_t* __restrict__ v0, const uint2* __restrict__ r0,
                              uint32_t* __restrict__ k1, uint32_t* __restrict__ v1, uint2* __restrict__ r1) {
    if (sctl[kSortWide] == 0u) return;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < M;
         i += (long long)gridDim.x * blockDim.x) {
        k1[i] = k0[i];
        v1[i] = v0[i];
        r1[i] = r0[i];
    }
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, long long n) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_f32(float* p, float v, long long n) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

unsigned grid_for(long long items, long long per_block, unsigned cap_blocks) {
    long long b = (items + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > cap_blocks) b = cap_blocks;
    return (unsigned)b;
}

// What the digits are counted from: no valid depth is below near_z.
uint32_t key_base(const Params& P) {
    uint32_t bits;
    memcpy(&bits, &P.near_z, sizeof(bits));
    return P.near_z > 0.0f ? bits : 0u;
}

// One stable LSD pass over the F segments of n elements; ping-pong is
// managed by the caller.
void radix_pass(int cur, int pass, const Params& P, const Workspace& w, hipStream_t s) {
    const long long n = P.n, tpf = w.max_sort_tiles;
    const int F = P.F, to = cur ^ 1;
    const uint32_t base = key_base(P);
    const unsigned tiles = (unsigned)(F * tpf), g = grid_for(tiles, 1, pass == kSortPasses ? 512 : 16384);
    {
        ProfScope _p("k_sort_upsweep", s);
        if (pass >= 2)
            hipLaunchKernelGGL(k_sort_upsweep<2>, dim3(g), dim3(kBigThreads), 0, s, w.dkey[cur], n, F, tpf, pass,
                               base, w.counts, w.sctl);
        else
            hipLaunchKernelGGL(k_sort_upsweep<1>, dim3(g), dim3(kBigThreads), 0, s, w.dkey[cur], n, F, tpf, pass,
                               base, w.counts, w.sctl);
    }
    {
        ProfScope _p("k_sort_scan", s);
        hipLaunchKernelGGL(k_sort_scan, dim3(kSortBuckets / kScanDigits, F), dim3(kScanDigits * kScanRuns), 0, s,
                           w.counts, (int)tpf, pass, w.totals, w.sctl);
    }
    {
        ProfScope _p("k_sort_downsweep", s);
        hipLaunchKernelGGL(k_sort_downsweep, dim3(tiles), dim3(kBigThreads), 0, s, w.dkey[cur],
                           pass ? w.dval[cur] : nullptr, w.drect[cur], w.dkey[to], w.dval[to], w.drect[to], n, tpf,
                           pass, base, w.counts, w.totals, w.sctl);
    }
}

}  // namespace

void launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    ProfScope _p("k_fill_u32", s);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n, 256 * 4, 4096)), dim3(256), 0, s, p, v,
                       (long long)n);
}

void launch_fill_f32(float* p, float v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    ProfScope _p("k_fill_f32", s);
    hipLaunchKernelGGL(k_fill_f32, dim3(grid_for(n, 256 * 4, 4096)), dim3(256), 0, s, p, v,
                       (long long)n);
}

void launch_depth_sort(const Params& P, const Workspace& w, hipStream_t s) {
    if (w.M == 0) return;
    int cur = 0;
    if (P.n <= kFrameSortMax) {
        static_assert(kFrameSortMax == 8 * kFrameThreads, "the largest frame a workgroup sorts");
        ProfScope _p("k_sort_frame", s);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(P.F), dim3(kFrameThreads), 0, s, w.dkey[0], w.drect[0], (uint32_t)P.n,
                               key_base(P), w.dkey[1], w.dval[1], w.drect[1]);
        };
        if (P.n <= 2 * kFrameThreads) go(k_sort_frame<2>);
        else if (P.n <= 4 * kFrameThreads) go(k_sort_frame<4>);
        else go(k_sort_frame<8>);
        return;
    }
    // the preprocess has cleared the control words (and shist for one sweep)
    if (one_sweep_sort(P, w)) {
        const long long tpf = w.max_sort_tiles;
        const unsigned tiles = (unsigned)(P.F * tpf);
        const uint32_t base = key_base(P);
        {
            ProfScope _p("k_sort_hist", s);
            hipLaunchKernelGGL(k_sort_hist, dim3(tiles), dim3(kSortThreads), 0, s, w.dkey[0], (long long)P.n,
                               tpf, base, w.shist, w.slook[0], w.sctl);
        }
        for (int pass = 0; pass <= kSortPasses; ++pass) {
            ProfScope _p("k_sort_onesweep", s);
            hipLaunchKernelGGL(k_sort_onesweep, dim3(tiles), dim3(kSortThreads), 0, s, w.dkey[cur],
                               pass ? w.dval[cur] : nullptr, w.drect[cur], w.dkey[cur ^ 1], w.dval[cur ^ 1],
                               w.drect[cur ^ 1], (long long)P.n, tpf, pass, base, w.shist, w.sctl, w.slook[pass & 1],
                               pass < kSortPasses ? w.slook[(pass + 1) & 1] : nullptr);
            cur ^= 1;
        }
        return;
    }
    for (int pass = 0; pass <= kSortPasses; ++pass, cur ^= 1) radix_pass(cur, pass, P, w, s);
}

void launch_sort_settle(const Workspace& w, hipStream_t s) {
    if (w.M == 0) return;
    hipLaunchKernelGGL(k_sort_settle, dim3(grid_for(w.M, 256, 4096)), dim3(256), 0, s, w.sctl, (long long)w.M,
                       w.dkey[0], w.dval[0], w.drect[0], w.dkey[1], w.dval[1], w.drect[1]);
}

}  // namespace gft
