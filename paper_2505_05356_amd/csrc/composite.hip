// Front-to-back compositing (forward) and back-to-front gradient recursion
// (backward) of RGB, mean depth and raw C-ToF quads, one workgroup per
// (frame, tile) work item: 1, 2 or 4 pixels per lane, by the batch's tiles.
//
// Forward (paper §3): for each pixel walk the tile's depth-sorted list and
//   alpha = min(alpha_max, o G(x)),  skip if alpha < alpha_min,
//   stop before compositing if T (1 - alpha) < T_min,
//   RGB += c alpha T (Eq. 2), D += d alpha T (Eq. 5),
//   S_f += a sin(psi_f) alpha T^2, C_f += a cos(psi_f) alpha T^2 (Eq. 4),
// then Q_{f,j} = cos(phi_j) S_f + sin(phi_j) C_f + q_bg T^p, because
// sin(psi + phi) = sin(psi) cos(phi) + cos(psi) sin(phi): two accumulators
// per frequency serve every phase offset.
//
// Backward (supplement C): walk the same list back to front from the last
// composited entry, recover T_k = T_{k+1} / (1 - alpha_k) from the saved
// T_final, and accumulate dL/dalpha_k with Eq. S2 (RGB, depth) and Eq. S3
// (quads) plus the background terms; then chain to the per-entry screen-space
// quantities.  Per-entry gradients are summed over the wave with DPP and
// added to the per-(frame, Gaussian) gradient record with one atomic per wave.
//
// Records of 64 list entries at a time are staged in LDS by each wave, in
// its own slice (the forward's waves walk their tile's list independently;
// the backward has one wave per tile in large batches and 2 or 4 waves, each
// with its own pixels, in small ones): one coalesced gather per entry of its
// 48-byte record and 16-byte conic, then every lane of the wave reads them as
// LDS broadcasts.  No MFMA: per (pixel, entry) this is ~20 FP32 VALU
// operations and one v_exp_f32.
#include <type_traits>

#include "block_scan.h"
#include "common.h"
#include "walk.h"

namespace gft {

namespace {

// Base-2 exponent q of the 2-D Gaussian at (px, py): the conic is stored
// prescaled by -log2(e) / 2 (-log2(e) for the cross term), so o G = o 2^q.
// One definition shared by the forward and the backward kernels, with
// contraction pinned, so both take identical skip / stop / clamp decisions:
// q = dy (C dy + B dx) + A dx^2, where the column terms B dx and A dx^2 are
// formed once per pixel column (splat_col) and reused by every pixel of it.
struct SplatCol {
    float dx, bdx, adx2;
};

__device__ __forceinline__ SplatCol splat_col(const float4 c, const float4 r1, float px) {
#pragma clang fp contract(off)
    SplatCol k;
    k.dx = px - c.x;
    k.bdx = r1.y * k.dx;
    k.adx2 = (r1.x * k.dx) * k.dx;
    return k;
}

__device__ __forceinline__ float splat_row(const SplatCol& k, const float4 c, const float4 r1, float py,
                                           float& dy) {
#pragma clang fp contract(off)
    dy = py - c.y;
    return __builtin_fmaf(dy, __builtin_fmaf(r1.z, dy, k.bdx), k.adx2);
}

// Below this exponent (log2 units) alpha < alpha_min with room to spare for
// the rounding of exp2, the product and the threshold itself.
constexpr float kSkipMargin = 1.0f / 64.0f;

// The staged form of an entry's centre for one tile: the centre relative to
// the tile origin (the hi + lo pair folded once per entry), and the exponent
// threshold thr with q < thr  =>  min(o 2^q, alpha_max) < alpha_min, which
// lets the backward skip an entry that no pixel of the tile can take without
// changing any decision.
// lamin = log2(alpha_min), or -inf when alpha_min = 0 (nothing skipped).
// The last slot is the caller's.
__device__ __forceinline__ float4 stage_centre(const float4 r0, float o, float ox, float oy, float lamin,
                                               float last = 0.f) {
    const float cu = (r0.x - ox) + r0.z;
    const float cv = (r0.y - oy) + r0.w;
    return make_float4(cu, cv, (lamin - __log2f(o)) - kSkipMargin, last);
}

// Pixel centres [x0, x1] x [y0, y1] relative to the tile origin.
struct PixelBox {
    float x0, x1, y0, y1;
};

// True only if no pixel of the box can take the entry: alpha < alpha_min at
// all of them, whatever the rounding.  The exponent's maximum over the box is
// 0 at the centre if the box holds it, else on an edge that faces the centre;
// err covers the rounding of this bound and of the pixels' own exponents.
// Anything that is not a number compares false, and the entry is kept.
__device__ __forceinline__ bool never_taken(const float4 c, const float4 r1, float lamin, const PixelBox& b) {
    const float dx0 = b.x0 - c.x, dx1 = b.x1 - c.x, dy0 = b.y0 - c.y, dy1 = b.y1 - c.y;
    const float ex = fminf(fmaxf(0.f, dx0), dx1), ey = fminf(fmaxf(0.f, dy0), dy1);
    const float hb = -0.5f * r1.y;
    const float ys = fminf(fmaxf(hb * ex * __builtin_amdgcn_rcpf(r1.z), dy0), dy1);
    const float xs = fminf(fmaxf(hb * ey * __builtin_amdgcn_rcpf(r1.x), dx0), dx1);
    const float qx = ys * (r1.z * ys + r1.y * ex) + r1.x * ex * ex;
    const float qy = ey * (r1.z * ey + r1.y * xs) + r1.x * xs * xs;
    const float mx = fmaxf(fabsf(dx0), fabsf(dx1)), my = fmaxf(fabsf(dy0), fabsf(dy1));
    const float err = 2e-6f * (fabsf(r1.x) * mx * mx + fabsf(r1.y) * mx * my + fabsf(r1.z) * my * my);
    const float thr = (lamin - __log2f(r1.w)) - kSkipMargin;
    return fmaxf(qx, qy) + err < thr && qx == qx && qy == qy;
}

// Sum over the 64 lanes of a wave: DPP within rows of 16, then 4 readlanes.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf,
                                                              0xf, true));
}

__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_f32<0xb1>(v);    // quad_perm [1,0,3,2]
    v += dpp_f32<0x4e>(v);    // quad_perm [2,3,0,1]
    v += dpp_f32<0x114>(v);   // row_shr:4
    v += dpp_f32<0x118>(v);   // row_shr:8 -> lane 15 of each row holds the row sum
    const int b = __builtin_bit_cast(int, v);
    return (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 15)) +
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 31))) +
           (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 47)) +
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 63)));
}

// Value of a lane whose index differs from this lane's in bit log2(D) and
// agrees in all higher bits (the lower ones may differ: the fold below goes
// from the high bits down, so they do not tell fields apart yet).
template <int D>
__device__ __forceinline__ float xchg(float x) {
    static_assert(D < 16, "rows of 16 lanes");
    if constexpr (D == 1) return dpp_f32<0xb1>(x);          // quad_perm [1,0,3,2]
    else if constexpr (D == 2) return dpp_f32<0x4e>(x);     // quad_perm [2,3,0,1]
    else if constexpr (D == 4) return dpp_f32<0x141>(x);    // row_half_mirror
    else return dpp_f32<0x128>(x);                          // row_ror:8
}

// Sum of a pair of fields over lane bit log2(D), each lane keeping one of
// them: a where its bit is 0, b where it is 1.  Across rows the swap
// instructions hand a's upper part against b's lower part, so the pair costs
// one swap and one add and no selects (an LDS permute with selects, four
// instructions and a round trip, before).  The two wait states before a swap
// cover operands that vector instructions have just written, which the
// compiler cannot see through the asm.
template <int D>
__device__ __forceinline__ float fold(float a, float b, int lane) {
    if constexpr (D == 32) {
        asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
        return a + b;
    } else if constexpr (D == 16) {
        asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
        return a + b;
    } else {
        const bool hi = (lane & D) != 0;
        const float send = hi ? a : b, keep = hi ? b : a;
        return keep + xchg<D>(send);
    }
}

// Reduce-scatter of N per-lane fields over the 64 lanes, one lane bit a
// level: pairs of fields fold into one register; the odd one is summed into
// both halves.  About 2 N instructions instead of 12 N for N reductions.
template <int N, int D = 32>
__device__ __forceinline__ float wave_reduce_fields(float (&v)[N], int lane) {
    if constexpr (D == 0) {
        static_assert(N == 1, "at most 64 fields");
        return v[0];
    } else {
        constexpr int H = (N + 1) / 2;
        float r[H];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) r[i] = fold<D>(v[2 * i], v[2 * i + 1], lane);
        if constexpr (N % 2 != 0) {
            if constexpr (D >= 16) r[H - 1] = fold<D>(v[N - 1], v[N - 1], lane);
            else r[H - 1] = v[N - 1] + xchg<D>(v[N - 1]);
        }
        return wave_reduce_fields<H, D / 2>(r, lane);
    }
}

// Field whose wave total this lane holds after wave_reduce_fields<N>, or -1
// if a lower lane holds the same one.
template <int N, int D = 32>
__device__ __forceinline__ int field_of_lane(int lane) {
    if constexpr (D == 0) {
        return 0;
    } else {
        const int r = field_of_lane<(N + 1) / 2, D / 2>(lane);
        const int bit = (lane & D) != 0 ? 1 : 0;
        if (r < 0) return -1;
        if (2 * r + 1 < N) return 2 * r + bit;
        return bit ? -1 : 2 * r;
    }
}

// The outputs of one pixel from its sums.
template <int NF>
__device__ __forceinline__ void write_pixel(const Params& P, const gftorf_frame& fr, const gftorf_outputs& out, int f,
                                            size_t HW, size_t pix, float cr, float cg, float cb, float dep,
                                            const float (&S)[NF], const float (&C)[NF], float T, uint32_t last) {
    if (out.rgb) {
        float* o = out.rgb + (size_t)f * 3 * HW + pix;
        o[0] = cr + fr.bg_rgb[0] * T;
        o[HW] = cg + fr.bg_rgb[1] * T;
        o[2 * HW] = cb + fr.bg_rgb[2] * T;
    }
    if (out.quad) {
        const float Tp = P.bg_pow == 2 ? T * T : T;
        float* o = out.quad + (size_t)f * P.nq * HW + pix;
#pragma unroll
        for (int i = 0; i < NF; ++i)
            for (int jj = 0; jj < P.nphi; ++jj) {
                const int qc = i * P.nphi + jj;
                if (fr.quad_mask == 0u || ((fr.quad_mask >> qc) & 1u))
                    o[qc * HW] = P.cphi[jj] * S[i] + P.sphi[jj] * C[i] + fr.bg_quad[qc] * Tp;
            }
    }
    if (out.phasor || out.d_tof || out.amplitude) {
        const float Tp = P.bg_pow == 2 ? T * T : T;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            float sh = 0.f, ch = 0.f;   // projections of the rendered quads (Eq. 1)
            for (int jj = 0; jj < P.nphi; ++jj) {
                const int qc = i * P.nphi + jj;
                const float q = P.cphi[jj] * S[i] + P.sphi[jj] * C[i] + fr.bg_quad[qc] * Tp;
                sh += P.cphi[jj] * q;
                ch += P.sphi[jj] * q;
            }
            const size_t o = ((size_t)f * P.nf + i) * HW + pix;
            if (out.phasor) {
                out.phasor[(((size_t)f * P.nf + i) * 2) * HW + pix] = ch;
                out.phasor[(((size_t)f * P.nf + i) * 2 + 1) * HW + pix] = sh;
            }
            if (out.d_tof) {
                float ph = atan2f(sh, ch);
                if (ph < 0.f) ph += 6.283185307179586f;
                out.d_tof[o] = (float)(kSpeedOfLight / (4.0 * M_PI * P.freq[i])) * ph;
            }
            if (out.amplitude) out.amplitude[o] = 0.5f * sqrtf(sh * sh + ch * ch);
        }
    }
    if (out.depth) out.depth[(size_t)f * HW + pix] = dep;
    out.T_final[(size_t)f * HW + pix] = T;
    out.n_contrib[(size_t)f * HW + pix] = (int32_t)last;
}

// Forward: WPT waves per (frame, tile), each walking the tile's list for its
// own pixels without a workgroup barrier; a lane owns PPT pixels of one column
// (pixel p = lane + 64 (wave + WPT i)).  The opacities of U consecutive
// entries do not depend on each other, so they are formed together; only the
// transmittance runs serially through them.
// Bound by vector instruction issue in large batches and by the length of one
// wave's instruction stream in small ones, so everything that is the same for
// a whole wave (who takes the entry, who stops, the workload counts) is kept
// as lane masks in scalar registers, and a wave only walks the entries that
// some pixel of its box may take: of those that its tile's list holds, 46% in
// an image of 64 x 48 pixels and 80% in the batches below.  One lane tests
// one entry while it is staged.  1M Gaussians x 16 frames 803 us with one
// pixel per lane in divergent branches, 645 with lane masks, 611 now; 200k x 8
// 172, 155, 142; one 640x480 frame of 100k 41, 38, 36; 12 tiles of 2k
// Gaussians 51, 48, 33.
template <int TW, int TH, int NF, int WPT, int U>
__global__ void __launch_bounds__(64 * WPT, WPT == 2 && NF <= 2 ? 6 : 1) k_composite_fwd(Params P, const gftorf_frame* __restrict__ frames,
                                                            const uint2* __restrict__ ranges,
                                                            const uint2* __restrict__ granges,
                                                            const uint32_t* __restrict__ gval,
                                                            const uint16_t* __restrict__ gloc,
                                                            uint32_t* __restrict__ tval,
                                                            uint8_t* __restrict__ touch,
                                                            const float4* __restrict__ rec,
                                                            const float4* __restrict__ conic,
                                                            gftorf_outputs out, uint2* __restrict__ wcount,
                                                            float* __restrict__ marks, uint32_t n_marks) {
    constexpr int PPT = TW * TH / (64 * WPT);
    static_assert(PPT * 64 * WPT == TW * TH && 64 % U == 0, "whole waves and groups of entries");
    constexpr int RS4 = record_float4s(NF);
    constexpr int SS4 = staged_float4s(NF);
    // 64 list entries are staged at a time (most pixels stop after 100-200, so
    // short batches waste few loads), by each wave for itself: those that some
    // pixel of its box may take, one after the other, then U that none takes.
    // SHARED: the workgroup's waves find the entries together.
    constexpr bool SHARED = WPT == 4;
    constexpr int NQ = SHARED ? 1 : WPT;
    __shared__ float4 srec_w[WPT][SS4][64 + U];
    // group-list entries of the tile found but not yet staged: fewer than a
    // batch, and one round of the walk more
    constexpr uint32_t QN = SHARED ? 2048 : 512;
    __shared__ uint32_t queue_w[NQ][QN];
    __shared__ uint32_t place_w[WPT][64];   // of a staged entry in its batch
    __shared__ uint32_t found_w[2][WPT], going_w[2][WPT];   // SHARED: per wave, by turn

    const int w = xcd_remap(blockIdx.x, gridDim.x);
    const int f = w / P.n_tiles;
    const int tile = w - f * P.n_tiles;
    const int ty = tile / P.ntx, tx = tile - ty * P.ntx;
    const int tid = threadIdx.x, lane = tid & 63;
    const int sub = __builtin_amdgcn_readfirstlane(tid / 64);
    const float ox = (float)(tx * TW), oy = (float)(ty * TH);
    const uint2 rg = ranges[w];
    const float amin = P.alpha_min, amax = P.alpha_max, tmin = P.T_min;

    // A wave's pixels form a box of BW x BH, as square as one column per lane
    // lets it be, so that many of its tile's entries miss it.
    constexpr int BW = TW == 32 && PPT > 1 ? 16 : 8, BH = 64 / BW * PPT, STEP = 64 / BW;
    static_assert(TW % BW == 0 && TH % BH == 0, "whole boxes");
    const int bx = sub % (TW / BW) * BW, by = sub / (TW / BW) * BH;
    const int px = bx + lane % BW, py = by + lane / BW;   // its pixels: (px, py + STEP i)
    const float lamin = amin > 0.f ? __log2f(amin) : -INFINITY;
    const PixelBox box = {(float)bx + 0.5f, (float)(bx + BW) - 0.5f, (float)by + 0.5f, (float)(by + BH) - 0.5f};
    // pixel centre relative to the tile origin (exact small values); a pixel
    // that has stopped (or lies outside) has an unreachable threshold
    const float fpx = (float)px + 0.5f;
    float fpy[PPT], T[PPT], cr[PPT], cg[PPT], cb[PPT], dep[PPT], S[PPT][NF], C[PPT][NF], thr[PPT];
    uint32_t last[PPT];
    uint64_t alive[PPT], any = 0ull;
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int row = py + STEP * i;
        fpy[i] = (float)row + 0.5f;
        T[i] = 1.0f;
        cr[i] = cg[i] = cb[i] = dep[i] = 0.f;
#pragma unroll
        for (int k = 0; k < NF; ++k) S[i][k] = C[i][k] = 0.f;
        const bool inside = tx * TW + px < P.W && ty * TH + row < P.H;
        thr[i] = inside ? amin : INFINITY;
        last[i] = 0;
        alive[i] = lanes(inside);
        any |= alive[i];
    }
    // evaluated / composited (pixel, entry) pairs of the wave: a pixel that
    // stops at entry e has evaluated e of them, one that never stops all
    uint32_t n_eval = 0, n_comp = 0;

    float4 (*srec)[64 + U] = srec_w[sub];
    uint32_t* place = place_w[sub];
    uint32_t* queue = queue_w[SHARED ? 0 : sub];
    auto sync = [] {   // LDS writes before this, reads after it, and the other way round
        if constexpr (SHARED) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };
    const uint32_t len = (uint32_t)__builtin_amdgcn_readfirstlane((int)(rg.y - rg.x));
    constexpr int NW = SHARED ? WPT : 1;
    TileWalk<NW> walk = tile_walk<NW>(P, f, tx, ty, granges, gloc, SHARED ? sub : 0, lane);
    uint32_t head = 0, queued = 0;   // of the queue
    uint32_t item = 0;               // this lane's of the next batch
    int turn = 0;
    auto next_items = [&] {
        while (queued < 64u && walk.more()) {
            const typename TileWalk<NW>::Hits h = walk.round();
            uint32_t tail = head + queued, all = h.count();
            if constexpr (SHARED) {
                if (lane == 0) found_w[turn][sub] = all;
                __syncthreads();
                all = 0;
#pragma unroll
                for (int q = 0; q < WPT; ++q) {
                    const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)found_w[turn][q]);
                    tail += q < sub ? n : 0u;
                    all += n;
                }
                turn ^= 1;
            }
            h.each([&](uint32_t entry, uint32_t q) { queue[(tail + q) % QN] = entry; });
            queued += all;
        }
        sync();
        if (lane < (int)queued) item = gval[queue[(head + lane) % QN]];
    };
    if (len != 0u) next_items();
    // some pixel of the wave (SHARED: of the tile, which has one inside the
    // image; its waves pass the same barriers, also one with no pixel inside)
    // has not stopped
    bool going = SHARED || any != 0ull;
    int cnt;
    for (uint32_t pos = 0; pos < len && going; pos += (uint32_t)cnt) {
        cnt = __builtin_amdgcn_readfirstlane((int)min(min(queued, 64u), len - pos));
        if (cnt == 0) break;   // the list is cut at the pair capacity
        if (pos != 0u && pos / 64u <= n_marks) {   // for the split backward; pos is a multiple of 64
            float* m = marks + ((size_t)w * n_marks + (pos / 64u - 1u)) * (TW * TH) + py * TW + px;
#pragma unroll
            for (int i = 0; i < PPT; ++i) m[STEP * TW * i] = T[i];
        }
        const bool have = lane < cnt;
        if (have && (!SHARED || sub == 0))
            tval[rg.x + pos + lane] = item;   // the backward walks the part that was composited
        const float4* r = rec + (size_t)item * RS4;
        float4 c = make_float4(0.f, 0.f, 0.f, 0.f), r1 = make_float4(0.f, 0.f, 0.f, -1.f);
        if (have) {
            c = r[0];
            r1 = conic[item];
        }
        c = make_float4((c.x - ox) + c.z, (c.y - oy) + c.w, 0.f, 0.f);
        const uint64_t hits = lanes(have) & ~lanes(never_taken(c, r1, lamin, box));
        const uint32_t slot = rank_below(hits), n_hits = (uint32_t)__popcll(hits);
        float4 fields[SS4 - 2];
#pragma unroll
        for (int q = 2; q < SS4; ++q) fields[q - 2] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (lane_of(hits))
#pragma unroll
            for (int q = 2; q < SS4; ++q) fields[q - 2] = r[q - 1];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // after the last batch's reads
        __builtin_amdgcn_wave_barrier();
        if (lane < U) {   // alpha = -1, below every threshold
            srec[0][n_hits + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
            srec[1][n_hits + lane] = make_float4(0.f, 0.f, 0.f, -1.f);
        }
        if (lane_of(hits)) {
            srec[0][slot] = c;
            srec[1][slot] = r1;
            place[slot] = (uint32_t)lane;
        }
        if constexpr (SHARED) __syncthreads();   // every wave has its items: the queue may be written
        head = (head + (uint32_t)cnt) % QN;
        queued -= (uint32_t)cnt;
        // the next batch's entries are found, and their items loaded, while
        // the rest of this one arrives and while it is walked
        const uint32_t walked = item;
        next_items();
        if (lane_of(hits))
#pragma unroll
            for (int q = 2; q < SS4; ++q) srec[q][slot] = fields[q - 2];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t pos0 = pos + 1u;   // list position of the batch's first entry
        constexpr uint32_t kStaged = 0x80000000u;   // `last` holds a staged entry's index
        uint32_t k0 = 0;
        for (; k0 < n_hits && any != 0ull; k0 += U) {
            float a[U][PPT];
            float4 fld[U][SS4 - 2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float4 c = srec[0][k0 + u], r1 = srec[1][k0 + u];
#pragma unroll
                for (int q = 2; q < SS4; ++q) fld[u][q - 2] = srec[q][k0 + u];
                const SplatCol col = splat_col(c, r1, fpx);
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    float dy;
                    a[u][i] = fminf(r1.w * __builtin_amdgcn_exp2f(splat_row(col, c, r1, fpy[i], dy)), amax);
                }
            }
            // formed here, not each where it is used behind a branch
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < PPT; ++i) asm volatile("" : "+v"(a[u][i]));
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    const float av = a[u][i];
                    const float nT = T[i] * (1.0f - av);
                    uint64_t take = lanes(av >= thr[i]);
                    const uint64_t stop = take & lanes(nT < tmin);   // stop before compositing
                    if (stop != 0ull) {
                        thr[i] = lane_of(stop) ? INFINITY : thr[i];
                        take &= ~stop;
                        alive[i] &= ~stop;
                        n_eval += (uint32_t)__popcll(stop) * (pos0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)place[k0 + u]));
                        any = 0ull;
#pragma unroll
                        for (int q = 0; q < PPT; ++q) any |= alive[q];
                    }
                    n_comp += (uint32_t)__popcll(take);
                    if (lane_of(take)) {
                        const float w1 = av * T[i];
                        const float w2 = w1 * T[i];
                        cr[i] += fld[u][0].x * w1;
                        cg[i] += fld[u][0].y * w1;
                        cb[i] += fld[u][0].z * w1;
                        dep[i] += fld[u][0].w * w1;
#pragma unroll
                        for (int k = 0; k < NF; ++k) {
                            const float4 rp = fld[u][1 + k / 2];
                            S[i][k] += ((k & 1) ? rp.z : rp.x) * w2;
                            C[i][k] += ((k & 1) ? rp.w : rp.y) * w2;
                        }
                        T[i] = nT;
                        last[i] = kStaged | (k0 + u);
                    }
                }
        }
#pragma unroll
        for (int i = 0; i < PPT; ++i)
            if (last[i] & kStaged) last[i] = pos0 + place[last[i] & 63u];
        // what no pixel walked has no gradient: the backward skips its record
        if (lane_of(hits) && slot < k0) touch[walked] = 1;
        going = any != 0ull;
        if constexpr (SHARED) {
            const int t = (int)(pos / 64u) & 1;
            if (lane == 0) going_w[t][sub] = going ? 1u : 0u;
            __syncthreads();
            uint32_t n = 0;
#pragma unroll
            for (int q = 0; q < WPT; ++q) n |= going_w[t][q];
            going = __builtin_amdgcn_readfirstlane((int)n) != 0;
        }
    }
#pragma unroll
    for (int i = 0; i < PPT; ++i) n_eval += (uint32_t)__popcll(alive[i]) * (rg.y - rg.x);
    {   // workload counters of this work item (algorithmic FLOP accounting);
        // summed over work items on the host by gftorf_read_status, not by
        // same-address atomics
        if constexpr (WPT == 1) {
            if (lane == 0) wcount[w] = make_uint2(n_eval, n_comp);
        } else {
            __shared__ uint2 wred[WPT];
            if (lane == 0) wred[sub] = make_uint2(n_eval, n_comp);
            __syncthreads();
            if (tid == 0) {
                uint2 t = wred[0];
                for (int q = 1; q < WPT; ++q) {
                    t.x += wred[q].x;
                    t.y += wred[q].y;
                }
                wcount[w] = t;
            }
        }
    }
    const gftorf_frame& fr = frames[f];
    const size_t HW = (size_t)P.H * P.W;
    for (int i = 0; i < PPT; ++i) {
        const int x = tx * TW + px, y = ty * TH + py + STEP * i;
        if (x < P.W && y < P.H)
            write_pixel<NF>(P, fr, out, f, HW, (size_t)y * P.W + x, cr[i], cg[i], cb[i], dep[i], S[i], C[i], T[i],
                            last[i]);
    }
}

// Backward: WPT waves per (frame, tile) (1 for large batches; 2 or 4 when
// the batch has too few tiles to fill the chip), each walking the tile's list
// for its own pixels; each lane owns PPT pixels of one column (pixel p = lane
// + 64 (wave + WPT i)), so the per-entry cross-lane reduction of the gradient
// fields is paid once for PPT pixels.
//
// The upstream gradients are constant per pixel, so the recursions of Eq. S2
// (RGB and depth, factor 1 - alpha) and Eq. S3 (quads, factor (1 - alpha)^2)
// only enter dL/dalpha through the per-entry values
//   u_k = sum_c dL/dc_c c_k,c + dL/dd d_k,  v_k = sum_f dL/dS_f a sin psi + dL/dC_f a cos psi
// and their suffix sums behind entry k, kept un-normalised:
//   A1 = sum_{j>k} u_j alpha_j T_j,  A2 = sum_{j>k} v_j alpha_j T_j^2.
// (The normalised accumulators of S2 / S3 are A1 / T_{k+1} and
// A2 / T_{k+1}^2.)  With the background term bg = c_bg . dL/dc T_final +
// p q_bg . dL/dq T_final^p,
//   dL/dalpha_k = T_k u_k + T_k^2 v_k - (A1 + 2 A2 + bg) / (1 - alpha_k),
// so one running sum A = A1 + 2 A2 + bg per pixel suffices:
//   A <- A + u_k alpha_k T_k + 2 v_k alpha_k T_k^2.
//
// SPLIT (batches of few tiles, whose waves would each walk a long list alone):
// the walk is cut into segments of whole 64-entry batches, a wave each.  The
// transmittance at a segment's end is the forward's own (marks); the suffix
// sum A there is the background term and the sums of u_j alpha_j T_j +
// 2 v_j alpha_j T_j^2 over the segments behind, which k_bwd_segment_sums forms
// first, walking them front to back: a third more arithmetic for a chain as
// long as one segment (where the line lies: kept_marks).

// One lane's pixels: constants of the walk and upstream gradients.
template <int NF, int PPT>
struct Pixels {
    float fpx, fpy[PPT];   // centres relative to the tile origin; the lane's pixels share a column
    uint32_t last[PPT];    // entries of the list up to the pixel's last composited one
    float gr[PPT][3], gd[PPT], gS[PPT][NF], gC[PPT][NF];
    float T_end[PPT], bg[PPT];   // final transmittance; background term of A
    uint32_t walk;         // largest `last` of the wave
};

template <int TW, int TH, int NF, int WPT, typename Bg>
__device__ __forceinline__ Pixels<NF, TW * TH / (64 * WPT)> load_pixels(
    const Params& P, const gftorf_frame& fr, int f, int tx, int ty, int sub, int lane,
    const float* __restrict__ T_final, const int32_t* __restrict__ n_contrib, const float* __restrict__ d_rgb,
    const float* __restrict__ d_quad, const float* __restrict__ d_depth, Bg bg_grad) {
    constexpr int PPT = TW * TH / (64 * WPT);
    Pixels<NF, PPT> px;
    const size_t HW = (size_t)P.H * P.W;
    px.fpx = (float)(lane % TW) + 0.5f;
    uint32_t walk = 0;
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int pidx = lane + 64 * (sub + WPT * i);
        const int x = tx * TW + pidx % TW, y = ty * TH + pidx / TW;
        const bool inside = x < P.W && y < P.H;
        px.fpy[i] = (float)(pidx / TW) + 0.5f;
        const size_t pix = (size_t)y * P.W + x;
        px.T_end[i] = 1.f;
        px.last[i] = 0;
        px.gr[i][0] = px.gr[i][1] = px.gr[i][2] = px.gd[i] = px.bg[i] = 0.f;
#pragma unroll
        for (int k = 0; k < NF; ++k) px.gS[i][k] = px.gC[i][k] = 0.f;
        if (inside) {
            // all loads are issued before any is used: a wave that is alone on
            // its SIMD would otherwise wait for each
            const float Tf = T_final[(size_t)f * HW + pix];
            px.last[i] = (uint32_t)n_contrib[(size_t)f * HW + pix];
            if (d_rgb)
                for (int c = 0; c < 3; ++c) px.gr[i][c] = d_rgb[((size_t)f * 3 + c) * HW + pix];
            if (d_depth) px.gd[i] = d_depth[(size_t)f * HW + pix];
            float q[NF][GFTORF_MAX_PHASE];
            if (d_quad)
#pragma unroll
                for (int k = 0; k < NF; ++k)
#pragma unroll
                    for (int jj = 0; jj < GFTORF_MAX_PHASE; ++jj)
                        q[k][jj] = d_quad[((size_t)f * P.nq + k * P.nphi + min(jj, P.nphi - 1)) * HW + pix];
            const float Tp = P.bg_pow == 2 ? Tf * Tf : Tf;
            float brd = 0.f, bqd = 0.f;
            for (int c = 0; c < 3; ++c) {
                brd += fr.bg_rgb[c] * px.gr[i][c];
                bg_grad(c, px.gr[i][c] * Tf);
            }
            if (d_quad)
#pragma unroll
                for (int k = 0; k < NF; ++k)
#pragma unroll
                    for (int jj = 0; jj < GFTORF_MAX_PHASE; ++jj) {
                        const int qc = k * P.nphi + jj;
                        // past the last phase, or a channel the frame does not render
                        if (jj >= P.nphi || (fr.quad_mask != 0u && !((fr.quad_mask >> qc) & 1u))) continue;
                        const float g = q[k][jj];
                        px.gS[i][k] += P.cphi[jj] * g;
                        px.gC[i][k] += P.sphi[jj] * g;
                        bqd += fr.bg_quad[qc] * g;
                        bg_grad(3 + GFTORF_MAX_PHASE * k + jj, g * Tp);
                    }
            px.T_end[i] = Tf;
            px.bg[i] = brd * Tf + (float)P.bg_pow * bqd * Tp;
        }
        walk = max(walk, px.last[i]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) walk = max(walk, (uint32_t)__shfl_xor((int)walk, o, 64));
    px.walk = (uint32_t)__builtin_amdgcn_readfirstlane((int)walk);
    return px;
}

// The segment `seg` of a wave's walk over `walk` list entries: runs of whole
// 64-entry batches that start at kept marks, as equal as their number allows,
// the last one to the end of the walk.
struct Segment {
    uint32_t n, beg, end;   // segments of the walk; list positions of this one
};

__device__ __forceinline__ Segment segment_of(uint32_t walk, uint32_t seg, uint32_t n_seg, uint32_t n_marks) {
    const uint32_t batches = min((walk + 63u) / 64u, n_marks + 1u);
    const uint32_t per = max(1u, (batches + n_seg - 1u) / n_seg);
    Segment s;
    s.n = max(1u, (batches + per - 1u) / per);
    s.beg = seg * per * 64u;
    s.end = seg + 1u >= s.n ? walk : (seg + 1u) * per * 64u;
    return s;
}

// Wave `b` of a split launch over `items` (tile, part of it) pairs: its item and
// segment.  Each XCD takes one contiguous eighth of the items, and inside it
// all first segments come before all second ones: many lists end in the first
// few, and with an item's segments side by side the round-robin dispatch would
// give some CUs only empty ones.
__device__ __forceinline__ bool split_item(uint32_t b, uint32_t items, uint32_t& item, uint32_t& seg) {
    const uint32_t per = (items + kXcds - 1u) / kXcds, i = b / kXcds;
    seg = i / per;
    item = b % kXcds * per + (i - seg * per);
    return item < items;
}
inline unsigned split_grid(int64_t items, int64_t segments) {
    return (unsigned)((items + kXcds - 1) / kXcds * kXcds * segments);
}

// The split walk's sums of u_j alpha_j T_j + 2 v_j alpha_j T_j^2 over each
// segment but the first, front to back from the kept transmittance.
template <int TW, int TH, int NF, int WPT, int U>
__global__ void __launch_bounds__(64) k_bwd_segment_sums(
    Params P, const gftorf_frame* __restrict__ frames, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ tval, const float4* __restrict__ rec, const float4* __restrict__ conic,
    const float* __restrict__ T_final, const int32_t* __restrict__ n_contrib, const float* __restrict__ d_rgb,
    const float* __restrict__ d_quad, const float* __restrict__ d_depth, const float* __restrict__ marks,
    float* __restrict__ seg_sums, uint32_t n_seg, uint32_t n_marks) {
    constexpr int PPT = TW * TH / (64 * WPT);
    constexpr int RS4 = record_float4s(NF);
    constexpr int SS4 = staged_float4s(NF);
    __shared__ float4 srec[SS4][64];
    uint32_t ws, seg;
    if (!split_item(blockIdx.x, (uint32_t)(P.F * P.n_tiles * WPT), ws, seg)) return;
    ++seg;   // the first segment's sum is not needed
    const int w = (int)ws / WPT, sub = (int)ws - w * WPT;
    const int f = w / P.n_tiles;
    const int tile = w - f * P.n_tiles;
    const int ty = tile / P.ntx, tx = tile - ty * P.ntx;
    const int lane = threadIdx.x;
    const uint2 rg = ranges[w];
    const Pixels<NF, PPT> px = load_pixels<TW, TH, NF, WPT>(P, frames[f], f, tx, ty, sub, lane, T_final, n_contrib,
                                                            d_rgb, d_quad, d_depth, [](int, float) {});
    const Segment sg = segment_of(min(px.walk, rg.y - rg.x), seg, n_seg, n_marks);
    if (seg >= sg.n) return;
    const float amin = P.alpha_min, amax = P.alpha_max;
    const float ox = (float)(tx * TW), oy = (float)(ty * TH);
    float T[PPT], A[PPT];
    const float* m = marks + ((size_t)w * n_marks + (sg.beg / 64u - 1u)) * (TW * TH) + lane + 64 * sub;
#pragma unroll
    for (int i = 0; i < PPT; ++i) T[i] = m[64 * WPT * i], A[i] = 0.f;
    for (uint32_t lo = sg.beg; lo < sg.end; lo += 64u) {
        const int cnt = (int)min(64u, sg.end - lo);
        __syncthreads();
        if (lane < cnt) {
            const uint32_t item = tval[rg.x + lo + lane];
            const float4* r = rec + (size_t)item * RS4;
            const float4 r0 = r[0];
            srec[0][lane] = make_float4((r0.x - ox) + r0.z, (r0.y - oy) + r0.w, 0.f, 0.f);
            srec[1][lane] = conic[item];
#pragma unroll
            for (int q = 1; q < RS4; ++q) srec[q + 1][lane] = r[q];
        }
        __syncthreads();
        for (int k0 = 0; k0 < cnt; k0 += U) {
            // entries past cnt are past every pixel's last: not taken
            float a[U][PPT];
#pragma unroll
            for (int e = 0; e < U; ++e) {
                const float4 c = srec[0][k0 + e], r1 = srec[1][k0 + e];
                const SplatCol col = splat_col(c, r1, px.fpx);
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    float dy;
                    a[e][i] = fminf(r1.w * __builtin_amdgcn_exp2f(splat_row(col, c, r1, px.fpy[i], dy)), amax);
                }
            }
#pragma unroll
            for (int e = 0; e < U; ++e) {
                const float4 r2 = srec[2][k0 + e];
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    const uint64_t take = lanes(lo + (uint32_t)(k0 + e) < px.last[i]) & lanes(a[e][i] >= amin);
                    if (lane_of(take)) {
                        const float u = px.gr[i][0] * r2.x + px.gr[i][1] * r2.y + px.gr[i][2] * r2.z + px.gd[i] * r2.w;
                        float v = 0.f;
#pragma unroll
                        for (int k = 0; k < NF; ++k) {
                            const float4 rp = srec[3 + k / 2][k0 + e];
                            const float t = px.gS[i][k] * ((k & 1) ? rp.z : rp.x) + px.gC[i][k] * ((k & 1) ? rp.w : rp.y);
                            v = k == 0 ? t : v + t;
                        }
                        const float x = T[i] * v;
                        A[i] += (a[e][i] * T[i]) * ((u + x) + x);
                        T[i] *= 1.0f - a[e][i];
                    }
                }
            }
        }
    }
    float* o = seg_sums + ((size_t)w * n_seg + seg) * (TW * TH) + lane + 64 * sub;
#pragma unroll
    for (int i = 0; i < PPT; ++i) o[64 * WPT * i] = A[i];
}

template <int TW, int TH, int NF, int WPT, bool SPLIT>
__global__ void __launch_bounds__(64) k_composite_bwd(
    Params P, const gftorf_frame* __restrict__ frames, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ tval, const float4* __restrict__ rec, const float4* __restrict__ conic,
    const float* __restrict__ T_final, const int32_t* __restrict__ n_contrib,
    const float* __restrict__ d_rgb, const float* __restrict__ d_quad, const float* __restrict__ d_depth,
    float* __restrict__ grec, float* __restrict__ d_bg, const float* __restrict__ marks,
    const float* __restrict__ seg_sums, uint32_t n_seg, uint32_t n_marks) {
    constexpr int PPT = TW * TH / (64 * WPT);   // pixels per lane
    constexpr int B = 64;                      // list entries staged per batch
    constexpr int RS4 = record_float4s(NF);
    constexpr int SS4 = staged_float4s(NF);
    constexpr int GS = grad_floats(NF);
    constexpr int NG = 10 + 2 * NF;            // gradient fields per entry
    __shared__ float4 srec[SS4][B];
    __shared__ uint32_t sitem[B];

    // the waves of a work item are consecutive after the remap: one XCD
    uint32_t ws, seg = 0u;
    if constexpr (SPLIT) {
        if (!split_item(blockIdx.x, (uint32_t)(P.F * P.n_tiles * WPT), ws, seg)) return;
    } else {
        ws = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    }
    const int w = (int)ws / WPT, sub = (int)ws - w * WPT;
    const int f = w / P.n_tiles;
    const int tile = w - f * P.n_tiles;
    const int ty = tile / P.ntx, tx = tile - ty * P.ntx;
    const int lane = threadIdx.x;
    const uint2 rg = ranges[w];
    const float amin = P.alpha_min, amax = P.alpha_max;
    const float lamin = amin > 0.f ? __log2f(amin) : -INFINITY;
    const float ox = (float)(tx * TW), oy = (float)(ty * TH);

    float bg_acc[3 + GFTORF_MAX_PHASE * NF];   // colour, then the phases of every frequency
#pragma unroll
    for (int c = 0; c < 3 + GFTORF_MAX_PHASE * NF; ++c) bg_acc[c] = 0.f;
    const Pixels<NF, PPT> px =
        load_pixels<TW, TH, NF, WPT>(P, frames[f], f, tx, ty, sub, lane, T_final, n_contrib, d_rgb, d_quad, d_depth,
                                     [&](int c, float v) { bg_acc[c] += v; });
    // background gradients: dL/dc_bg = sum d_rgb T_final, dL/dq_bg = sum d_quad T_final^p
    if (d_bg && seg == 0u) {
#pragma unroll
        for (int c = 0; c < 3 + GFTORF_MAX_PHASE * NF; ++c) {
            const int k = (c - 3) / GFTORF_MAX_PHASE, jj = (c - 3) % GFTORF_MAX_PHASE;
            if (c >= 3 && jj >= P.nphi) continue;
            const float v = wave_sum(bg_acc[c]);
            if (lane == 0 && v != 0.f)
                atomicAdd(&d_bg[(size_t)f * (3 + P.nq) + (c < 3 ? c : 3 + k * P.nphi + jj)], v);
        }
    }
    Segment sg{1u, 0u, min(px.walk, rg.y - rg.x)};
    if constexpr (SPLIT) {
        sg = segment_of(sg.end, seg, n_seg, n_marks);
        if (seg >= sg.n) return;
    }
    // the state behind the segment; the suffix sum starts with the background term
    float T[PPT], A[PPT];
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        T[i] = px.T_end[i];
        A[i] = px.bg[i];
    }
    if constexpr (SPLIT) {
        const int p0 = lane + 64 * sub;
        if (seg + 1u < sg.n) {
            const float* m = marks + ((size_t)w * n_marks + (sg.end / 64u - 1u)) * (TW * TH) + p0;
#pragma unroll
            for (int i = 0; i < PPT; ++i) T[i] = m[64 * WPT * i];
        }
        for (uint32_t q = sg.n; q-- > seg + 1u;) {
            const float* m = seg_sums + ((size_t)w * n_seg + q) * (TW * TH) + p0;
#pragma unroll
            for (int i = 0; i < PPT; ++i) A[i] += m[64 * WPT * i];
        }
    }
    // the record field this lane adds to, and its constant factor: the exponent
    // is in log2 units, and the centre's terms lack -2
    const int fld = field_of_lane<NG>(lane);
    const float LN2 = 0.6931471805599453f;
    const float fscale = fld == 0 || fld == 1 ? -2.0f * LN2 : fld < 5 ? LN2 : 1.0f;

    const uint32_t first = rg.x + sg.beg;
    for (uint32_t hi = rg.x + sg.end; hi > first; ) {
        const uint32_t lo = (hi - first > (uint32_t)B) ? hi - B : first;
        const int cnt = (int)(hi - lo);
        __syncthreads();
        if (lane < cnt) {
            const uint32_t item = tval[hi - 1 - lane];
            sitem[lane] = item;
            const float4* r = rec + (size_t)item * RS4;
            const float4 r1 = conic[item];
            // 1 / o turns sum gq into d/do (0 where o is too small for either)
            srec[0][lane] = stage_centre(r[0], r1.w, ox, oy, lamin, r1.w > 1e-30f ? 1.0f / r1.w : 0.f);
            srec[1][lane] = r1;
#pragma unroll
            for (int q = 1; q < RS4; ++q) srec[q + 1][lane] = r[q];
        }
        __syncthreads();
        // the centre and conic of the next entry are read while this one is
        // taken (a wave alone on its SIMD otherwise waits for LDS each time)
        float4 cn = srec[0][0], r1n = srec[1][0];
        for (int s = 0; s < cnt; ++s) {
            const uint32_t kidx = hi - 1 - (uint32_t)s - rg.x;   // position in the tile list
            const float4 c = cn, r1 = r1n;
            cn = srec[0][(s + 1) & (B - 1)];
            r1n = srec[1][(s + 1) & (B - 1)];
            // phase 1: which pixels can composite this entry (the forward's
            // decisions: not past the pixel's last entry, exponent above the
            // certain-skip threshold); an entry no pixel takes costs no more
            float dy[PPT], qe[PPT];
            uint64_t pass[PPT], anyp = 0ull;
            const SplatCol col = splat_col(c, r1, px.fpx);   // the lane's pixels share a column
#pragma unroll
            for (int i = 0; i < PPT; ++i) {
                qe[i] = splat_row(col, c, r1, px.fpy[i], dy[i]);
                pass[i] = lanes(kidx < px.last[i]) & ~lanes(qe[i] < c.z);
                anyp |= pass[i];
            }
            if (anyp == 0ull) continue;
            const float4 r2 = srec[2][s];
            float as[NF], ac[NF];
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                const float4 rp = srec[3 + k / 2][s];
                as[k] = (k & 1) ? rp.z : rp.x;
                ac[k] = (k & 1) ? rp.w : rp.y;
            }
            // Sums start from their first term (pixel 0), not from 0 + term:
            // the compiler must keep an addition of +0 (it turns -0 into +0)
            float g[NG];
            auto put = [](float& acc, float term, int i) { acc = i == 0 ? term : acc + term; };
            uint64_t any = 0ull;
            // Branch-free per pixel: inactive pixels contribute zero and keep
            // their state (selects instead of divergent blocks, so the field
            // registers are never copied at control-flow joins).
            // The conic, centre and opacity gradients only need, per lane (one
            // pixel column, so one dx), sum gq, sum gq dy and sum gq dy^2, with
            // gq = dL/dq / ln 2 = o G dL/dalpha
            float p0, p1, p2;
            // alpha = o 2^q unless clamped at alpha_max, where it has no
            // gradient; an entry with o <= alpha_max never is (2^q <= 1 but for
            // the rounding of q, which the margin covers)
            auto pixels = [&](auto clamps) {
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    const float oG = r1.w * __builtin_amdgcn_exp2f(qe[i]);
                    const float a = decltype(clamps)::value ? fminf(oG, amax) : oG;
                    const uint64_t act = pass[i] & lanes(a >= amin);
                    any |= act;
                    // ae = alpha of a composited entry, 0 otherwise: with ae = 0
                    // every state update below is the identity (rcp(1) = 1)
                    const float ae = lane_of(act) ? a : 0.0f;
                    const float rom = __builtin_amdgcn_rcpf(1.0f - ae);
                    const float Ti = T[i] * rom;
                    const float u = px.gr[i][0] * r2.x + px.gr[i][1] * r2.y + px.gr[i][2] * r2.z + px.gd[i] * r2.w;
                    float v = px.gS[i][0] * as[0] + px.gC[i][0] * ac[0];
#pragma unroll
                    for (int k = 1; k < NF; ++k) v += px.gS[i][k] * as[k] + px.gC[i][k] * ac[k];
                    const float x = Ti * v, y = u + x;
                    const float dA = Ti * y - rom * A[i];
                    T[i] = Ti;
                    const float w1 = ae * Ti;
                    const float w2 = w1 * Ti;
                    A[i] += w1 * (y + x);
                    put(g[6], w1 * px.gr[i][0], i);
                    put(g[7], w1 * px.gr[i][1], i);
                    put(g[8], w1 * px.gr[i][2], i);
                    put(g[9], w1 * px.gd[i], i);
#pragma unroll
                    for (int k = 0; k < NF; ++k) {
                        put(g[10 + 2 * k], w2 * px.gS[i][k], i);
                        put(g[11 + 2 * k], w2 * px.gC[i][k], i);
                    }
                    const float aq = decltype(clamps)::value && oG > amax ? 0.0f : ae;
                    const float gq = dA * aq;
                    const float gy = gq * dy[i];
                    put(p0, gq, i);
                    put(p1, gy, i);
                    put(p2, gy * dy[i], i);
                }
            };
            if (__builtin_amdgcn_readfirstlane((int)(r1.w > 0.9999f * amax)))
                pixels(std::true_type{});
            else
                pixels(std::false_type{});
            if (any == 0ull) continue;
            {
                const float gx = col.dx * p0;                    // sum gx; sum gy = p1
                const float hb = 0.5f * r1.y;
                g[0] = r1.x * gx + hb * p1;                      // d/du: -(2 cA sum gx + cB sum gy)
                g[1] = r1.z * p1 + hb * gx;                      // d/dv: -(2 cC sum gy + cB sum gx)
                g[2] = col.dx * gx;                              // d/dcA
                g[3] = col.dx * p1;                              // d/dcB
                g[4] = p2;                                       // d/dcC
                g[5] = p0;                                       // d/do o
            }
            // one reduce-scatter over the wave, then one atomic instruction whose
            // lanes add consecutive fields of the entry's gradient record
            const float tot = wave_reduce_fields<NG>(g, lane) * (fld == 5 ? c.w : fscale);
            if (fld >= 0 && tot != 0.f) atomicAdd(grec + (size_t)sitem[s] * GS + fld, tot);
        }
        hi = lo;
    }
}


template <int TW, int TH, int WPT, int U>
hipError_t fwd_wpt(const Params& P, const gftorf_frame* frames, const Workspace& w, const gftorf_outputs& out,
                   hipStream_t s) {
    const unsigned blocks = (unsigned)(P.F * P.n_tiles);
#define GFT_FWD(NF_)                                                                                          \
    hipLaunchKernelGGL((k_composite_fwd<TW, TH, NF_, WPT, U>), dim3(blocks), dim3(64 * WPT), 0, s, P, frames, \
                       w.ranges, w.granges, w.gval, w.gloc, w.tval, w.touch, w.rec, w.conic, out, w.wcount, w.marks, (uint32_t)kept_marks((int64_t)P.F * P.n_tiles, TW * TH))
    switch (P.nf) {
        case 1: GFT_FWD(1); break;
        case 2: GFT_FWD(2); break;
        case 3: GFT_FWD(3); break;
        default: GFT_FWD(4); break;
    }
#undef GFT_FWD
    return hipGetLastError();
}

// Batches of fewer tiles than this take one pixel per lane and groups of four
// entries (more waves, and the longest chain each wave can hide), larger ones
// two pixels per lane and groups of two (the column's terms and the staging
// shared).  Measured: 1200 tiles 35.8 against 42.0 us, 2400 tiles 55.2 against
// 54.0, 3600 tiles 74.2 against 71.6, 4800 tiles 92 against 85, 9600 tiles 167
// against 141.
constexpr int64_t kFwdTiles = 2048;

template <int TW, int TH>
hipError_t fwd_nf(const Params& P, const gftorf_frame* frames, const Workspace& w,
                  const gftorf_outputs& out, hipStream_t s) {
    ProfScope _p("k_composite_fwd", s);
    if constexpr (TW * TH >= 256) {
        if ((int64_t)P.F * P.n_tiles < kFwdTiles) return fwd_wpt<TW, TH, 4, 4>(P, frames, w, out, s);
        return fwd_wpt<TW, TH, 2, 2>(P, frames, w, out, s);
    } else {
        return fwd_wpt<TW, TH, 1, 4>(P, frames, w, out, s);
    }
}

template <int TW, int TH, int WPT, bool SPLIT>
hipError_t bwd_wpt(const Params& P, const gftorf_frame* frames, const Workspace& w,
                   const gftorf_outputs& sv, const float* dr, const float* dq, const float* dd,
                   float* dbg, hipStream_t s) {
    const int64_t tiles = (int64_t)P.F * P.n_tiles;
    const uint32_t marks = (uint32_t)kept_marks(tiles, TW * TH);
    const uint32_t segs = SPLIT ? (uint32_t)split_segments(tiles, TW * TH) : 1u;
    const unsigned waves = (unsigned)(tiles * WPT);
    constexpr int U = TW * TH / (64 * WPT) == 1 ? 4 : 2;
#define GFT_BWD(NF_)                                                                                          \
    if constexpr (SPLIT) {                                                                                    \
        ProfScope _p("k_bwd_segment_sums", s);                                                                \
        hipLaunchKernelGGL((k_bwd_segment_sums<TW, TH, NF_, WPT, U>), dim3(split_grid(waves, segs - 1u)), dim3(64), 0, \
                           s, P, frames, w.ranges, w.tval, w.rec, w.conic, sv.T_final, sv.n_contrib, dr, dq,  \
                           dd, w.marks, w.seg_sums, segs, marks);                                             \
    }                                                                                                         \
    {                                                                                                         \
        ProfScope _p("k_composite_bwd", s);                                                                   \
        hipLaunchKernelGGL((k_composite_bwd<TW, TH, NF_, WPT, SPLIT>), dim3(SPLIT ? split_grid(waves, segs) : waves), dim3(64), 0, s, P, \
                           frames, w.ranges, w.tval, w.rec, w.conic, sv.T_final, sv.n_contrib, dr, dq, dd,    \
                           w.grec, dbg, w.marks, w.seg_sums, segs, marks);                                    \
    }
    switch (P.nf) {
        case 1: GFT_BWD(1); break;
        case 2: GFT_BWD(2); break;
        case 3: GFT_BWD(3); break;
        default: GFT_BWD(4); break;
    }
#undef GFT_BWD
    return hipGetLastError();
}

template <int TW, int TH>
hipError_t bwd_nf(const Params& P, const gftorf_frame* frames, const Workspace& w,
                  const gftorf_outputs& sv, const float* dr, const float* dq, const float* dd,
                  float* dbg, hipStream_t s) {
    const int64_t tiles = (int64_t)P.F * P.n_tiles;
    if (kept_marks(tiles, TW * TH) == 0) return bwd_wpt<TW, TH, 1, false>(P, frames, w, sv, dr, dq, dd, dbg, s);
    if constexpr (TW * TH >= 256) {
        const int wpt = split_waves(tiles, TW * TH);
        if (wpt == 4) return bwd_wpt<TW, TH, 4, true>(P, frames, w, sv, dr, dq, dd, dbg, s);
        if (wpt == 2) return bwd_wpt<TW, TH, 2, true>(P, frames, w, sv, dr, dq, dd, dbg, s);
    }
    return bwd_wpt<TW, TH, 1, true>(P, frames, w, sv, dr, dq, dd, dbg, s);
}

}  // namespace

hipError_t launch_composite_fwd(const Params& P, const gftorf_frame* frames, const Workspace& w,
                                const gftorf_outputs& out, hipStream_t s) {
    if (P.tw == 8 && P.th == 8) return fwd_nf<8, 8>(P, frames, w, out, s);
    if (P.tw == 32 && P.th == 8) return fwd_nf<32, 8>(P, frames, w, out, s);
    return fwd_nf<16, 16>(P, frames, w, out, s);
}

hipError_t launch_composite_bwd(const Params& P, const gftorf_frame* frames, const Workspace& w,
                                const gftorf_outputs& saved, const float* d_rgb,
                                const float* d_quad, const float* d_depth, float* d_bg,
                                hipStream_t s) {
    if (P.tw == 8 && P.th == 8) return bwd_nf<8, 8>(P, frames, w, saved, d_rgb, d_quad, d_depth, d_bg, s);
    if (P.tw == 32 && P.th == 8) return bwd_nf<32, 8>(P, frames, w, saved, d_rgb, d_quad, d_depth, d_bg, s);
    return bwd_nf<16, 16>(P, frames, w, saved, d_rgb, d_quad, d_depth, d_bg, s);
}

}  // namespace gft
