// Deformation network of paper §4 ("MLP") on the gfx950 matrix cores.
//
// delta x = W_8 h_8 + b_8,  h_{l+1} = relu(W_l h_l + b_l),  h_0 = the positional
// encoding of (s_x x0, s_t t), for every (time, Gaussian) row.
//
// Kernels
//   k_mlp_pack    float32 parameters -> bfloat16 weight copies: W_l as
//                 [out][in] (forward) and W_l^T as [in][out] (backward), both
//                 zero-padded so every product is whole 16 x 16 x 32 tiles.
//   k_mlp_fwd     one workgroup of 4 waves per 128 rows: the encoding and
//                 every layer's activations stay in LDS (128 x 256 bf16),
//                 weights stream from L2, two k-steps ahead; wave w computes
//                 output features 64w .. 64w+63 of all 128 rows with
//                 v_mfma_f32_16x16x32_bf16, the weights as the A operand.
//                 Two workgroups share a CU (two waves per SIMD), so one's
//                 epilogue overlaps the other's products.  Training mode also
//                 stores h_0 .. h_8 and the ReLU decisions as bits.
//   k_mlp_bwd     the same tiling backwards: gz_8 = dL/d delta, then per layer
//                 g_l = gz_l W_l, gz_{l-1} = g_l * [h_l > 0] (the forward's
//                 bits); stores every gz_l and, from g_0, the gradient of the
//                 scaled centre input.  Two workgroups per CU, as the forward.
//   k_mlp_dw      dW_l = sum_rows gz_l h_l^T, db_l = sum_rows gz_l: rows are the
//                 contraction, split into fixed chunks, one partial per chunk;
//                 each 64-row stage of gz_l and h_l passes once through LDS,
//                 which transposes the fragments as they are read.
//   k_mlp_reduce  sums the chunk partials in chunk order into the parameter
//                 layout; k_mlp_dx0 sums the centre gradient over the times.
//   k_blend       Eq. 7 with the network: per-frame offsets from the offsets
//                 at two integer timesteps; k_blend_bwd is its transpose.
//
// With the weights as the A operand a lane holds four consecutive features of
// a row, so the epilogues write LDS by 8 bytes (32 writes per layer and lane
// instead of 128 of 2 bytes) and the ReLU and its bits cost 8 instructions per
// four elements (16 before).  Activations and gradients are saved row-major,
// as LDS holds them, by whole cache lines and past L2 (non-temporal), where
// the weights stay.  Loads and stores retire in order, so the two k-steps of
// weights that the next layer starts with are loaded before the stores.
// 1.6M rows: forward 2.09 -> 1.92 ms (without saves 1.47 -> 1.37 ms, 1.13
// PFLOP/s, where a large library product reaches 1.20 on the same card),
// backward 2.49 -> 2.36 ms.  What is left of both is the stores: 1.3 ms
// alone, at the rate of a plain fill, and 1.7 ms the products alone.
//
// The forward also keeps the ReLU decisions of h_1 .. h_8 as bits, 16 bytes
// per lane and layer in the lane's own accumulator order, so the backward
// gates its gradients from 4 registers instead of re-reading the activations.
#include <mutex>

#include "mlp.h"

namespace gft {
namespace mlp {
namespace {

// Scratch of gftorf_mlp_fwd_noalloc: the bfloat16 weight copies of one
// inference forward.  Every GPU the library runs on holds its own copy until
// the process ends.  In host code this name is only a stand-in for the
// symbol: kernels receive the device address that noalloc_scratch resolves.
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

// Third word of a raw buffer descriptor (32-bit untyped elements).
constexpr int kBufferWord3 = 0x00020000;

// LDS row stride in bf16: the 16-byte pad puts the 16 rows of one fragment
// read in 16 distinct 4-bank groups.
constexpr int kLDX = kWidth + 8;

struct Args {
    const float* x0;
    int64_t n, rows;
    int lx, lt;
    float sx, st;
    float times[kMaxTimes];
    const gftorf_frame* frames;   // if set, time t is frames[t].time (device)
    const bf16* wf[kLayers];
    const bf16* wt[kLayers];
    const float* bias[kLayers];
    bf16* H[kLayers];
    bf16* GZ[kLayers];
    uint4* mask;   // [blocks][kDepth][256 threads]: word c, bit mask_bit(r, j) = [h > 0] of acc[r][c][j]
};

// D += A B on one 16 x 16 tile, K = 32.  Lane l supplies A[l % 16][8 (l / 16) + e]
// and B[8 (l / 16) + e][l % 16], e = 0..7; it receives D[4 (l / 16) + j][l % 16].
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Positional encoding, the network's input features: of the scaled centre p
// the blocks p, sin(2^k pi p), cos(2^k pi p), k = 0 .. lx - 1, of its three
// coordinates, then the same of the scaled time.

__device__ __forceinline__ float pick4(const float (&v)[4], int c) {
    return c == 0 ? v[0] : c == 1 ? v[1] : c == 2 ? v[2] : v[3];
}

// scaled inputs of row r (zeros for padding rows)
__device__ __forceinline__ void row_inputs(const Args& a, int64_t r, float (&xin)[4]) {
    xin[0] = xin[1] = xin[2] = xin[3] = 0.f;
    if (r >= a.rows) return;
    const int t = (int)(r / a.n);
    const int64_t k = r - (int64_t)t * a.n;
    for (int c = 0; c < 3; ++c) xin[c] = a.sx * a.x0[c * a.n + k];
    xin[3] = a.st * (a.frames ? a.frames[t].time : a.times[t]);
}

// acc[r][c] += W[col0 + 16 c + .][.] * X[16 r + .][.]^T over K: X in LDS
// (row-major, stride kLDX), W in global memory as [features][K].  The weights
// are the A operand, so a lane receives four consecutive features of one row
// (row 16 r + l % 16, features col0 + 16 c + 4 (l / 16) + j), which it writes
// back to LDS and gates with 8-byte accesses.
// The next k-step's weight fragments are in flight while this one multiplies
// (pinned by a scheduling barrier).
// `w` holds the first D k-steps' weight fragments (first_weights), which the
// caller loads before the previous layer's stores.
template <int K, int D>
__device__ __forceinline__ void first_weights(const bf16* __restrict__ W, int col0, bf16x8 (&w)[D][4], int lane) {
    const bf16* wp = W + (size_t)(col0 + (lane & 15)) * K + (lane >> 4) * 8;
#pragma unroll
    for (int d = 0; d < D && 32 * d < K; ++d)
#pragma unroll
        for (int c = 0; c < 4; ++c) w[d][c] = *(const bf16x8*)(wp + (size_t)16 * c * K + 32 * d);
}

template <int K, int D>
__device__ __forceinline__ void gemm_128x64(const bf16* X, const bf16* __restrict__ W, int col0,
                                            f32x4 (&acc)[8][4], bf16x8 (&w)[D][4], int lane) {
    const int lr = lane & 15, lk = (lane >> 4) * 8;
    const bf16* wp = W + (size_t)(col0 + lr) * K + lk;
    bf16x8 wn[4];
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 32) {
        if (k0 + 32 * D < K) {
#pragma unroll
            for (int c = 0; c < 4; ++c) wn[c] = *(const bf16x8*)(wp + (size_t)16 * c * K + k0 + 32 * D);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const bf16x8 x = *(const bf16x8*)(X + (16 * r + lr) * kLDX + lk + k0);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[r][c] = mfma(w[0][c], x, acc[r][c]);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int d = 0; d + 1 < D; ++d) w[d][c] = w[d + 1][c];
            if (k0 + 32 * D < K) w[D - 1][c] = wn[c];
        }
    }
}

// Writes the first K columns of the LDS rows to `dst`, row-major [128][K],
// between a product that reads them and the barrier after it: the stores
// complete under the epilogue, and no weight load waits behind them (loads and
// stores retire in order).  K / 8 lanes write a row's 16-byte pieces, so whole
// cache lines leave together.
template <int K>
__device__ __forceinline__ void save_rows(const bf16* X, bf16* __restrict__ dst, int tid) {
    constexpr int P = K / 8, N = 128 * P / 256;   // pieces per row, and per thread
    // four in flight, none of them hoisted into the product (whose registers
    // leave no room), and one lane offset for all of them (buffer addressing)
    __builtin_amdgcn_sched_barrier(0);
    const __amdgpu_buffer_rsrc_t out =
        __builtin_amdgcn_make_buffer_rsrc(dst, 0, 128 * K * (int)sizeof(bf16), kBufferWord3);
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q0 = 0; q0 < N; q0 += 4) {
        u32x4 v[4];
#pragma unroll
        for (int q = q0; q < q0 + 4 && q < N; ++q) {
            const int i = tid + 256 * q;
            v[q - q0] = *(const u32x4*)(X + i / P * kLDX + i % P * 8);
        }
#pragma unroll
        for (int q = q0; q < q0 + 4 && q < N; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(v[q - q0], out, 16 * tid, 16 * 256 * q, 2);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Two float32 to a packed pair of bfloat16, round to nearest even.
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// Bit of element j of accumulator row tile r in its column tile's mask word.
// The forward takes the four bits of a tile from the two 32-bit words of its
// bfloat16 ReLU outputs (each half a non-negative int16, non-zero if active):
// the smaller of each half and 1, the second word's beside the first's.
__device__ __forceinline__ constexpr int mask_bit(int r, int j) { return 2 * r + (j >> 1) + 16 * (j & 1); }

__device__ __forceinline__ uint32_t relu_bits(uint2 v, int r) {
    // (as an instruction: the compiler would make two compares and selects of it)
    uint32_t lo, hi;
    asm("v_pk_min_i16 %0, %1, %2" : "=v"(lo) : "v"(v.x), "s"(0x00010001));
    asm("v_pk_min_i16 %0, %1, %2" : "=v"(hi) : "v"(v.y), "s"(0x00010001));
    return (lo | (hi << 1)) << (2 * r);
}

__device__ __forceinline__ void zero(f32x4 (&acc)[8][4]) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
}

template <bool SAVE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_mlp_fwd(Args a, float* __restrict__ delta) {
    __shared__ __attribute__((aligned(16))) bf16 X[kRows * kLDX];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * kRows;
    {   // h_0: two threads per row, each every other frequency (sine and cosine
        // from one reduction); the coordinates themselves and the padding by both
        const int rr = tid >> 1, half = tid & 1;
        float xin[4];
        row_inputs(a, r0 + rr, xin);
        bf16* h = X + rr * kLDX;
        const int nx = 3 * (1 + 2 * a.lx);
        for (int k = half; k < a.lx; k += 2)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                float sn, cs;
                sincospif(ldexpf(xin[c], k), &sn, &cs);   // 2^k p is exact
                h[3 * (1 + 2 * k) + c] = (bf16)sn;
                h[3 * (2 + 2 * k) + c] = (bf16)cs;
            }
        for (int k = half; k < a.lt; k += 2) {
            float sn, cs;
            sincospif(ldexpf(xin[3], k), &sn, &cs);
            h[nx + 1 + 2 * k] = (bf16)sn;
            h[nx + 2 + 2 * k] = (bf16)cs;
        }
        if (half == 0) {
            for (int c = 0; c < 3; ++c) h[c] = (bf16)xin[c];
            h[nx] = (bf16)xin[3];
        } else {
            for (int f = nx + 1 + 2 * a.lt; f < kK0; ++f) h[f] = (bf16)0.f;
        }
    }
    __syncthreads();
    f32x4 acc[8][4];
    const int col0 = 64 * wv;
    bf16x8 w[2][4];
    first_weights<kK0>(a.wf[0], col0, w, lane);
    auto bias = [&](int l) {   // the products accumulate onto the bias
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float* bb = a.bias[l] + col0 + 16 * c + 4 * lg;
            const f32x4 bv = {bb[0], bb[1], bb[2], bb[3]};
#pragma unroll
            for (int r = 0; r < 8; ++r) acc[r][c] = bv;
        }
    };
    auto activate = [&](int l) {   // h_{l+1} = relu(acc), into LDS
        __syncthreads();   // every wave has read this layer's input
        uint32_t mw[4] = {0u, 0u, 0u, 0u};
        bf16* xo = X + lr * kLDX + col0 + 4 * lg;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                // bfloat16 first, then ReLU as a packed 16-bit integer max with 0:
                // a negative bfloat16 is a negative int16
                uint2 v = make_uint2(pack2(acc[r][c][0], acc[r][c][1]), pack2(acc[r][c][2], acc[r][c][3]));
                asm("v_pk_max_i16 %0, %1, 0" : "=v"(v.x) : "v"(v.x));
                asm("v_pk_max_i16 %0, %1, 0" : "=v"(v.y) : "v"(v.y));
                *(uint2*)(xo + 16 * r * kLDX + 16 * c) = v;
                if (SAVE) mw[c] |= relu_bits(v, r);
            }
        }
        if (SAVE) a.mask[((size_t)blockIdx.x * kDepth + l) * 256 + tid] = make_uint4(mw[0], mw[1], mw[2], mw[3]);
        __syncthreads();
    };
    bias(0);
    gemm_128x64<kK0>(X, a.wf[0], col0, acc, w, lane);
    first_weights<kWidth>(a.wf[1], col0, w, lane);
    if (SAVE) save_rows<kK0>(X, a.H[0] + (size_t)r0 * kK0, tid);
    activate(0);
    for (int l = 1; l < kDepth; ++l) {
        bias(l);
        gemm_128x64<kWidth>(X, a.wf[l], col0, acc, w, lane);
        if (l + 1 < kDepth) first_weights<kWidth>(a.wf[l + 1], col0, w, lane);
        if (SAVE) save_rows<kWidth>(X, a.H[l] + (size_t)r0 * kWidth, tid);
        activate(l);
    }
    // head: 16 (3 real) outputs x 128 rows; wave w takes rows 32w .. 32w+31
    f32x4 o2[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    const bf16* bp = a.wf[kDepth] + (size_t)lr * kWidth + 8 * lg;
#pragma unroll 4
    for (int k0 = 0; k0 < kWidth; k0 += 32) {
        const bf16x8 b = *(const bf16x8*)(bp + k0);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const bf16x8 x = *(const bf16x8*)(X + (32 * wv + 16 * r + lr) * kLDX + 8 * lg + k0);
            o2[r] = mfma(b, x, o2[r]);
        }
    }
    if (SAVE) save_rows<kWidth>(X, a.H[kDepth] + (size_t)r0 * kWidth, tid);
    if (lg == 0) {   // the lane's first four outputs of its row: three are real
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int64_t row = r0 + 32 * wv + 16 * r + lr;
            if (row < a.rows) {
                const int t = (int)(row / a.n);
                const int64_t k = row - (int64_t)t * a.n;
#pragma unroll
                for (int j = 0; j < 3; ++j) delta[((int64_t)t * 3 + j) * a.n + k] = o2[r][j] + a.bias[kDepth][j];
            }
        }
    }
}

// The ReLU decisions of the training forward as plain bytes, dec[row][layer][unit]
// (1 = active), read from (WRITE = false) or written into (WRITE = true) the
// bit words: one thread per word, i.e. per (128-row block, layer, forward
// thread), which holds the thread's 4 column tiles x 8 row tiles x 4 features.
// Padding rows read nothing and are written inactive.
template <bool WRITE>
__global__ void __launch_bounds__(256) k_mlp_decisions(uint4* __restrict__ mask, uint8_t* __restrict__ dec,
                                                       int64_t rows, int64_t words) {
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (w >= words) return;
    const int tid = (int)(w & 255);
    const int l = (int)((w >> 8) % kDepth);
    const int64_t blk = (w >> 8) / kDepth;
    const int lane = tid & 63, wv = tid >> 6, lr = lane & 15, lg = lane >> 4;
    uint32_t mw[4] = {0u, 0u, 0u, 0u};
    if (!WRITE) {
        const uint4 m = mask[w];
        mw[0] = m.x, mw[1] = m.y, mw[2] = m.z, mw[3] = m.w;
    }
    for (int c = 0; c < 4; ++c) {
        for (int r = 0; r < 8; ++r)
            for (int j = 0; j < 4; ++j) {
                const int64_t row = blk * kRows + 16 * r + lr;
                if (row >= rows) continue;
                uint8_t* d = dec + (row * kDepth + l) * kWidth + 64 * wv + 16 * c + 4 * lg + j;
                if (WRITE)
                    mw[c] |= (*d != 0 ? 1u : 0u) << mask_bit(r, j);
                else
                    *d = (uint8_t)((mw[c] >> mask_bit(r, j)) & 1u);
            }
    }
    if (WRITE) mask[w] = make_uint4(mw[0], mw[1], mw[2], mw[3]);
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_mlp_bwd(Args a, const float* __restrict__ d_delta,
                                                 float* __restrict__ dxr) {
    __shared__ __attribute__((aligned(16))) bf16 X[kRows * kLDX];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * kRows;
    {   // gz_8 = dL/d delta of the block's rows, padded to kHeadK columns
        const int rr = tid >> 1, half = tid & 1;
        const int64_t r = r0 + rr;
        float g[4] = {0.f, 0.f, 0.f, 0.f};
        if (r < a.rows) {
            const int t = (int)(r / a.n);
            const int64_t k = r - (int64_t)t * a.n;
            for (int c = 0; c < 3; ++c) g[c] = d_delta[((int64_t)t * 3 + c) * a.n + k];
        }
        for (int c = 16 * half; c < 16 * half + 16; ++c)
            X[rr * kLDX + c] = (bf16)(c < 3 ? pick4(g, c) : 0.f);
    }
    __syncthreads();
    // two threads per row: its 16 padded columns
    *(bf16x8*)(a.GZ[kDepth] + (size_t)(r0 + (tid >> 1)) * kOutPad + 8 * (tid & 1)) =
        *(const bf16x8*)(X + (tid >> 1) * kLDX + 8 * (tid & 1));

    f32x4 acc[8][4];
    const int col0 = 64 * wv;
    // the forward's ReLU decisions for h_{l+1} (layer l's output), loaded
    // before the product so that their latency hides behind it
    uint4 hm;
    auto load_masks = [&](int l) { hm = a.mask[((size_t)blockIdx.x * kDepth + l) * 256 + tid]; };
    load_masks(kDepth - 1);
    zero(acc);
    bf16x8 w[2][4];
    first_weights<kHeadK>(a.wt[kDepth], col0, w, lane);
    gemm_128x64<kHeadK>(X, a.wt[kDepth], col0, acc, w, lane);   // g_8 = gz_8 W_8
    first_weights<kWidth>(a.wt[kDepth - 1], col0, w, lane);
    for (int l = kDepth - 1; l >= 0; --l) {
        __syncthreads();
        // gz_l = g_{l+1} * [h_{l+1} > 0]
        const uint32_t mw[4] = {hm.x, hm.y, hm.z, hm.w};
        bf16* xo = X + lr * kLDX + col0 + 4 * lg;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                // bfloat16 first, then the gates as 16-bit masks: shifting the
                // word puts the bits of elements (0, 1), then (2, 3), at bits 15
                // and 31, and an arithmetic shift of each half by 15 spreads them
                uint2 z = make_uint2(pack2(acc[r][c][0], acc[r][c][1]), pack2(acc[r][c][2], acc[r][c][3]));
                z.x &= __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, mw[c] << (15 - 2 * r)) >> (short)15);
                z.y &= __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, mw[c] << (14 - 2 * r)) >> (short)15);
                *(uint2*)(xo + 16 * r * kLDX + 16 * c) = z;
            }
        }
        __syncthreads();
        if (l > 0) {
            load_masks(l - 1);
            zero(acc);
            gemm_128x64<kWidth>(X, a.wt[l], col0, acc, w, lane);   // g_l = gz_l W_l
            if (l > 1) first_weights<kWidth>(a.wt[l - 1], col0, w, lane);
            save_rows<kWidth>(X, a.GZ[l] + (size_t)r0 * kWidth, tid);
        }
    }
    // g_0 = gz_0 W_0 -> [128][96]: wave w takes rows 32w .. 32w+31, all 6 column tiles
    f32x4 g0[2][6];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 6; ++c) g0[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
        const bf16* bp = a.wt[0] + (size_t)lr * kWidth + 8 * lg;
#pragma unroll 2
        for (int k0 = 0; k0 < kWidth; k0 += 32) {
            bf16x8 b[6];
#pragma unroll
            for (int c = 0; c < 6; ++c) b[c] = *(const bf16x8*)(bp + (size_t)16 * c * kWidth + k0);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const bf16x8 x = *(const bf16x8*)(X + (32 * wv + 16 * r + lr) * kLDX + 8 * lg + k0);
#pragma unroll
                for (int c = 0; c < 6; ++c) g0[r][c] = mfma(b[c], x, g0[r][c]);
            }
        }
    }
    save_rows<kWidth>(X, a.GZ[0] + (size_t)r0 * kWidth, tid);
    __syncthreads();
    constexpr int kLDF = kK0 + 4;   // float stride of g_0 in LDS
    float* XF = reinterpret_cast<float*>(X);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 6; ++c)
            *(f32x4*)(XF + (32 * wv + 16 * r + lr) * kLDF + 16 * c + 4 * lg) = g0[r][c];
    __syncthreads();
    {   // d(scaled centre) = sum over the x features of g_0 * d enc / d p; two threads per row
        const int rr = tid >> 1, half = tid & 1;
        const int64_t r = r0 + rr;
        float xin[4];
        row_inputs(a, r, xin);
        const float* g = XF + rr * kLDF;
        float s[3] = {0.f, 0.f, 0.f};
        if (half == 0)
            for (int c = 0; c < 3; ++c) s[c] = g[c];
        for (int k = half; k < a.lx; k += 2) {
            const float w = ldexpf(3.14159265358979f, k);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                float sn, cs;
                sincospif(ldexpf(xin[c], k), &sn, &cs);
                s[c] += g[3 * (1 + 2 * k) + c] * (w * cs) - g[3 * (2 + 2 * k) + c] * (w * sn);
            }
        }
        float s0 = s[0], s1 = s[1], s2 = s[2];
        s0 += __shfl_xor(s0, 1, 64);
        s1 += __shfl_xor(s1, 1, 64);
        s2 += __shfl_xor(s2, 1, 64);
        if (half == 0 && r < a.rows) {
            dxr[r * 3 + 0] = a.sx * s0;
            dxr[r * 3 + 1] = a.sx * s1;
            dxr[r * 3 + 2] = a.sx * s2;
        }
    }
}

// dW_l [NO][NI] and db_l [NO] of one row chunk.  8 waves: OG groups of output
// rows times IG groups of input columns; each wave keeps MT x NT tiles.
struct DwArgs {
    const bf16* GZ[kLayers];
    const bf16* H[kLayers];
    int64_t part_off[kLayers];
    int64_t part_stride, rows_pad, rows_per_chunk;
    float* part;
};

// bf16 of one staged row, padded to a stride that puts eight consecutive
// rows' 32 bytes in distinct banks
__host__ __device__ constexpr int staged_row(int features) { return features + (features % 32 == 16 ? 0 : 16); }
constexpr int dw_lds(int no, int ni) { return 2 * 64 * (staged_row(no) + staged_row(ni)); }   // two stages

// NO x NI of the FO x FI weights of layer l, from output oo and input ii.
template <int NO, int NI, int OG, int IG, int FO, int FI>
__device__ __forceinline__ void dw_chunk(const DwArgs& d, int l, int oo, int ii, bf16* lds) {
    constexpr int MT = NO / 16 / OG, NT = NI / 16 / IG;
    static_assert(OG * IG == 8 && MT * 16 * OG == NO && NT * 16 * IG == NI, "tiling");
    // One stage is two k-steps of 32 rows of gz (NO features) and h (NI
    // features), row-major as saved: staged once per workgroup in LDS,
    // double-buffered, and read from there by the 8 waves (each gradient tile
    // is read by IG waves and each activation tile by OG).  The contraction
    // runs over the rows, so the fragments are transposed as they are read
    // (ds_read_b64_tr_b16: four rows of 16 features, a lane per feature).
    constexpr int SO = staged_row(NO), SI = staged_row(NI);
    static_assert(SO / 2 % 16 == 8 && SI / 2 % 16 == 8, "row strides of an odd number of 8-bank steps");
    constexpr int CO = NO / 8, CI = NI / 8;           // 16-byte chunks per row
    constexpr int NC = 64 * (CO + CI);
    constexpr int PER = (NC + 511) / 512;
    auto sbuf = [&](int b) { return lds + b * (64 * (SO + SI)); };
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const int o0 = (wv / IG) * MT * 16, i0 = (wv % IG) * NT * 16;
    const bf16* __restrict__ GZ = d.GZ[l] + oo;
    const bf16* __restrict__ H = d.H[l] + ii;
    const int64_t rs = (int64_t)blockIdx.x * d.rows_per_chunk;
    const int64_t re = min(rs + d.rows_per_chunk, d.rows_pad);   // both multiples of 64
    const int nk = rs < re ? (int)((re - rs) / 64) : 0;          // stages; chunks hold multiples of 64 rows
    f32x4 acc[MT][NT];
    // db on the matrix cores: the product with a fragment of ones sums every
    // output row over the chunk's rows (the waves of the first input group)
    f32x4 ab[MT];
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.0f;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        ab[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // chunk q < 64 CO: gz row q / CO, features 8 (q % CO) ..; else h likewise
    bf16x8 stg[PER];
    auto fetch = [&](int64_t row) {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int q = tid + 512 * p;
            if (q < NC) {
                if (q < 64 * CO) {
                    // whole rows are one run of chunks
                    const size_t at = NO == FO ? (size_t)q * 8 : (size_t)(q / CO) * FO + q % CO * 8;
                    stg[p] = *(const bf16x8*)(GZ + (size_t)row * FO + at);
                } else {
                    const int qh = q - 64 * CO;
                    const size_t at = NI == FI ? (size_t)qh * 8 : (size_t)(qh / CI) * FI + qh % CI * 8;
                    stg[p] = *(const bf16x8*)(H + (size_t)row * FI + at);
                }
            }
        }
    };
    auto stage = [&](int b) {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int q = tid + 512 * p;
            if (q < NC) {
                const int qh = q - 64 * CO;
                const int at = q < 64 * CO ? q / CO * SO + q % CO * 8 : 64 * SO + qh / CI * SI + qh % CI * 8;
                *(bf16x8*)(sbuf(b) + at) = stg[p];
            }
        }
    };
    // this lane's fragment of 16 features from f0 over 32 rows: rows 4 lg .. +3
    // and 16 + 4 lg .. +3, the same order for both operands
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    auto fragment = [&](const bf16* s0, int stride, int f0) {
        const bf16* at = s0 + (4 * lg + (lr >> 2)) * stride + f0 + 4 * (lr & 3);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + 16 * stride));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    if (nk > 0) {
        fetch(rs);
        stage(0);
    }
    __syncthreads();
    for (int k = 0; k < nk; ++k) {
        const int cur = k & 1;
        const bool more = k + 1 < nk;
        if (more) fetch(rs + 64 * (k + 1));   // in flight during this stage's products
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 av[MT], bv[NT];
#pragma unroll
            for (int m = 0; m < MT; ++m) av[m] = fragment(sbuf(cur) + 32 * h * SO, SO, o0 + 16 * m);
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[t] = fragment(sbuf(cur) + 64 * SO + 32 * h * SI, SI, i0 + 16 * t);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[m][t] = mfma(av[m], bv[t], acc[m][t]);
            if (ii + i0 == 0)
#pragma unroll
                for (int m = 0; m < MT; ++m) ab[m] = mfma(av[m], ones, ab[m]);
        }
        if (more) stage(cur ^ 1);   // the other buffer was last read before the previous barrier
        __syncthreads();
    }
    float* P = d.part + (int64_t)blockIdx.x * d.part_stride + d.part_off[l];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                P[(size_t)(oo + o0 + 16 * m + 4 * lg + j) * FI + ii + i0 + 16 * t + lr] = acc[m][t][j];
    if (ii + i0 == 0 && lr == 0) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) P[(size_t)FO * FI + oo + o0 + 16 * m + 4 * lg + j] = ab[m][j];
    }
}

// The seven square layers (grid y).
__global__ void __launch_bounds__(512) k_mlp_dw(DwArgs d) {
    __shared__ __attribute__((aligned(16))) bf16 lds[dw_lds(kWidth, kWidth)];
    dw_chunk<kWidth, kWidth, 4, 2, kWidth, kWidth>(d, 1 + blockIdx.y, 0, 0, lds);
}

// The input layer and the head, each in two halves (grid y): 576 workgroups
// of which two share a CU.  With one workgroup per chunk and layer, in two
// launches, 112 of the 256 CUs were idle: 507 us for 1.6M rows.
__global__ void __launch_bounds__(512) k_mlp_dw_ends(DwArgs d) {
    __shared__ __attribute__((aligned(16))) bf16 lds[dw_lds(kWidth / 2, kK0)];
    static_assert(dw_lds(kOutPad, kWidth / 2) <= dw_lds(kWidth / 2, kK0), "the head's stages fit");
    const int half = (blockIdx.y & 1) * (kWidth / 2);
    if (blockIdx.y < 2) dw_chunk<kWidth / 2, kK0, 4, 2, kWidth, kK0>(d, 0, half, 0, lds);
    else dw_chunk<kOutPad, kWidth / 2, 1, 8, kOutPad, kWidth>(d, kDepth, 0, half, lds);
}

struct RedArgs {
    int64_t off_w[kLayers], off_b[kLayers], part_off[kLayers];
    int out[kLayers], in[kLayers];
    int64_t n_params, part_stride;
    int n_chunks;
};

// parameter gradient = sum of the chunk partials, chunk 0 first
__global__ void __launch_bounds__(256) k_mlp_reduce(RedArgs r, const float* __restrict__ part,
                                                    float* __restrict__ d_params) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= r.n_params) return;
    int l = 0;
    while (l + 1 < kLayers && p >= r.off_w[l + 1]) ++l;
    int64_t src;
    if (p < r.off_b[l]) {
        const int64_t e = p - r.off_w[l];
        const int o = (int)(e / r.in[l]), i = (int)(e - (int64_t)o * r.in[l]);
        src = r.part_off[l] + (int64_t)o * pad_in(l) + i;
    } else {
        src = r.part_off[l] + (int64_t)pad_out(l) * pad_in(l) + (p - r.off_b[l]);
    }
    // eight partials loaded at a time, added in chunk order
    float s = 0.f;
    int c = 0;
    for (; c + 8 <= r.n_chunks; c += 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = part[(int64_t)(c + j) * r.part_stride + src];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; c < r.n_chunks; ++c) s += part[(int64_t)c * r.part_stride + src];
    d_params[p] = s;
}

__global__ void __launch_bounds__(256) k_mlp_dx0(const float* __restrict__ dxr, int64_t n, int T,
                                                 int accumulate, float* __restrict__ d_x0) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f;
    for (int t = 0; t < T; ++t) {
        const float* g = dxr + ((int64_t)t * n + k) * 3;
        s0 += g[0];
        s1 += g[1];
        s2 += g[2];
    }
    if (accumulate) {
        s0 += d_x0[k];
        s1 += d_x0[n + k];
        s2 += d_x0[2 * n + k];
    }
    d_x0[k] = s0;
    d_x0[n + k] = s1;
    d_x0[2 * n + k] = s2;
}

struct PackArgs {
    int64_t off_w[kLayers];
    int out[kLayers], in[kLayers];
    bf16* wf[kLayers];
    bf16* wt[kLayers];
};

__global__ void __launch_bounds__(256) k_mlp_pack(PackArgs p, const float* __restrict__ params) {
    const int l = blockIdx.y;
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int out = p.out[l], in = p.in[l];
    const float* W = params + p.off_w[l];
    const int NO = pad_out(l), NI = pad_in(l), KO = pad_k(l);
    if (e < NO * NI) {
        const int o = e / NI, i = e - o * NI;
        p.wf[l][e] = (bf16)((o < out && i < in) ? W[(int64_t)o * in + i] : 0.f);
    }
    if (e < NI * KO) {
        const int i = e / KO, o = e - i * KO;
        p.wt[l][e] = (bf16)((o < out && i < in) ? W[(int64_t)o * in + i] : 0.f);
    }
}

// Eq. 7 weights of a frame (1, 0 without anchors)
__device__ __forceinline__ void eq7_weights(const gftorf_frame& fr, float& w1, float& w2) {
    if (fr.t_hi > fr.t_lo) {
        const float span = fr.t_hi - fr.t_lo;
        w1 = (fr.t_hi - fr.time) / span;
        w2 = (fr.time - fr.t_lo) / span;
    } else {
        w1 = 1.0f;
        w2 = 0.0f;
    }
}

// out[f] = w1_f steps[lo_f] + w2_f steps[hi_f], one thread per (frame, element)
__global__ void __launch_bounds__(256) k_blend(Blend b, const float* __restrict__ steps,
                                               const gftorf_frame* __restrict__ frames,
                                               float* __restrict__ out) {
    const int64_t per = 3 * b.n;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)b.n_frames * per) return;
    const int f = (int)(i / per);
    const int64_t e = i - (int64_t)f * per;
    float w1, w2;
    eq7_weights(frames[f], w1, w2);
    float v = w1 * steps[(int64_t)b.anchors[2 * f] * per + e];
    if (w2 != 0.0f) v += w2 * steps[(int64_t)b.anchors[2 * f + 1] * per + e];
    out[i] = v;
}

// d_steps[s] = sum over frames (in frame order) of the weight of s times d_frames[f]
__global__ void __launch_bounds__(256) k_blend_bwd(Blend b, const float* __restrict__ d_frames,
                                                   const gftorf_frame* __restrict__ frames,
                                                   float* __restrict__ d_steps) {
    const int64_t per = 3 * b.n;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)b.n_steps * per) return;
    const int st = (int)(i / per);
    const int64_t e = i - (int64_t)st * per;
    float acc = 0.0f;
    for (int f = 0; f < b.n_frames; ++f) {
        const int lo = b.anchors[2 * f], hi = b.anchors[2 * f + 1];
        if (lo != st && hi != st) continue;
        float w1, w2;
        eq7_weights(frames[f], w1, w2);
        const float g = d_frames[(int64_t)f * per + e];
        if (lo == st) acc += w1 * g;
        if (hi == st && w2 != 0.0f) acc += w2 * g;
    }
    d_steps[i] = acc;
}

Args make_args(const Layout& L, const Call& c) {
    Args a;
    a.x0 = c.x0;
    a.n = L.n;
    a.rows = L.rows;
    a.lx = L.lx;
    a.lt = L.lt;
    a.sx = c.sx;
    a.st = c.st;
    for (int t = 0; t < kMaxTimes; ++t) a.times[t] = t < L.n_times ? c.times[t] : 0.f;
    a.frames = c.frames;
    for (int l = 0; l < kLayers; ++l) {
        a.wf[l] = reinterpret_cast<const bf16*>(c.ws + L.wf[l]);
        a.wt[l] = reinterpret_cast<const bf16*>(c.ws + L.wt[l]);
        a.bias[l] = c.params + L.off_b[l];
        a.H[l] = L.training ? reinterpret_cast<bf16*>(c.ws + L.H[l]) : nullptr;
        a.GZ[l] = L.training ? reinterpret_cast<bf16*>(c.ws + L.GZ[l]) : nullptr;
    }
    a.mask = L.training ? reinterpret_cast<uint4*>(c.ws + L.mask) : nullptr;
    return a;
}

}  // namespace

hipError_t noalloc_scratch(char** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static char* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p || reinterpret_cast<uintptr_t>(p) % 256) return hipErrorInvalidValue;
        addr[dev] = static_cast<char*>(p);
    }
    *out = addr[dev];
    return hipSuccess;
}

bool make_layout(int lx, int lt, int width, int depth, int64_t n, int n_times, bool training,
                 Layout* L) {
    if (width != kWidth || depth != kDepth || lx < 0 || lt < 0 || n < 1 || n_times < 1 ||
        n_times > kMaxTimes)
        return false;
    const int n_in = 3 * (1 + 2 * lx) + 1 + 2 * lt;
    if (n_in > kK0 || n > (int64_t(1) << 40) / n_times) return false;
    L->lx = lx;
    L->lt = lt;
    L->n_in = n_in;
    int64_t off = 0;
    for (int l = 0; l < kLayers; ++l) {
        L->out[l] = l == kDepth ? 3 : kWidth;
        L->in[l] = l == 0 ? n_in : kWidth;
        L->off_w[l] = off;
        off += (int64_t)L->out[l] * L->in[l];
        L->off_b[l] = off;
        off += L->out[l];
    }
    L->n_params = off;
    L->n = n;
    L->n_times = n_times;
    L->rows = n * n_times;
    L->rows_pad = (L->rows + kRows - 1) / kRows * kRows;
    int64_t rpc = (L->rows_pad + kMaxChunks - 1) / kMaxChunks;
    rpc = (rpc + 63) / 64 * 64;   // whole 64-row stages of the weight-gradient kernel
    L->rows_per_chunk = rpc;
    L->n_chunks = (int)((L->rows_pad + rpc - 1) / rpc);
    int64_t po = 0;
    for (int l = 0; l < kLayers; ++l) {
        L->part_off[l] = po;
        po += (int64_t)pad_out(l) * pad_in(l) + pad_out(l);
    }
    L->part_stride = po;
    size_t b = 0;
    auto take = [&](size_t bytes) {
        const size_t at = b;
        b += (bytes + 255) / 256 * 256;
        return at;
    };
    for (int l = 0; l < kLayers; ++l) {
        L->wf[l] = take((size_t)pad_out(l) * pad_in(l) * 2);
        L->wt[l] = take((size_t)pad_in(l) * pad_k(l) * 2);
    }
    for (int l = 0; l < kLayers; ++l) L->H[l] = L->GZ[l] = 0;
    L->mask = L->dxr = L->part = 0;
    if (training) {
        for (int l = 0; l < kLayers; ++l) L->H[l] = take((size_t)L->rows_pad * pad_in(l) * 2);
        for (int l = 0; l < kLayers; ++l) L->GZ[l] = take((size_t)L->rows_pad * pad_out(l) * 2);
        // ReLU bits: 16 bytes per thread, layer and 128-row block = 2 bytes per row and unit
        L->mask = take((size_t)(L->rows_pad / kRows) * kDepth * 256 * 16);
        L->dxr = take((size_t)L->rows_pad * 3 * 4);
        L->part = take((size_t)L->n_chunks * L->part_stride * 4);
    }
    L->bytes = b;
    L->training = training;
    return true;
}

hipError_t launch_fwd(const Layout& L, const Call& c, float* delta, bool save, hipStream_t s) {
    PackArgs p;
    for (int l = 0; l < kLayers; ++l) {
        p.off_w[l] = L.off_w[l];
        p.out[l] = L.out[l];
        p.in[l] = L.in[l];
        p.wf[l] = reinterpret_cast<bf16*>(c.ws + L.wf[l]);
        p.wt[l] = reinterpret_cast<bf16*>(c.ws + L.wt[l]);
    }
    {
        ProfScope _p("k_mlp_pack", s);
        hipLaunchKernelGGL(k_mlp_pack, dim3(kWidth * kWidth / 256, kLayers), dim3(256), 0, s, p, c.params);
    }
    const Args a = make_args(L, c);
    const unsigned blocks = (unsigned)(L.rows_pad / kRows);
    ProfScope _f("k_mlp_fwd", s);
    if (save)
        hipLaunchKernelGGL(k_mlp_fwd<true>, dim3(blocks), dim3(256), 0, s, a, delta);
    else
        hipLaunchKernelGGL(k_mlp_fwd<false>, dim3(blocks), dim3(256), 0, s, a, delta);
    return hipGetLastError();
}

hipError_t launch_blend(const Blend& b, const float* steps, const gftorf_frame* frames, float* out,
                        hipStream_t s) {
    const int64_t total = (int64_t)b.n_frames * 3 * b.n;
    if (total == 0) return hipSuccess;
    ProfScope _p("k_blend", s);
    hipLaunchKernelGGL(k_blend, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, b, steps, frames, out);
    return hipGetLastError();
}

hipError_t launch_blend_bwd(const Blend& b, const float* d_frames, const gftorf_frame* frames,
                            float* d_steps, hipStream_t s) {
    const int64_t total = (int64_t)b.n_steps * 3 * b.n;
    if (total == 0) return hipSuccess;
    ProfScope _p("k_blend_bwd", s);
    hipLaunchKernelGGL(k_blend_bwd, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, b, d_frames,
                       frames, d_steps);
    return hipGetLastError();
}

hipError_t launch_bwd(const Layout& L, const Call& c, const float* d_delta, float* d_params,
                      float* d_x0, bool accumulate_x0, hipStream_t s) {
    const Args a = make_args(L, c);
    float* dxr = reinterpret_cast<float*>(c.ws + L.dxr);
    {
        ProfScope _b("k_mlp_bwd", s);
        hipLaunchKernelGGL(k_mlp_bwd, dim3((unsigned)(L.rows_pad / kRows)), dim3(256), 0, s, a,
                           d_delta, dxr);
    }
    DwArgs d;
    for (int l = 0; l < kLayers; ++l) {
        d.GZ[l] = a.GZ[l];
        d.H[l] = a.H[l];
        d.part_off[l] = L.part_off[l];
    }
    d.part_stride = L.part_stride;
    d.rows_pad = L.rows_pad;
    d.rows_per_chunk = L.rows_per_chunk;
    d.part = reinterpret_cast<float*>(c.ws + L.part);
    {
        ProfScope _w("k_mlp_dw", s);
        const unsigned nc = (unsigned)L.n_chunks;
        hipLaunchKernelGGL(k_mlp_dw, dim3(nc, kDepth - 1), dim3(512), 0, s, d);
        hipLaunchKernelGGL(k_mlp_dw_ends, dim3(nc, 4), dim3(512), 0, s, d);
    }
    RedArgs r;
    for (int l = 0; l < kLayers; ++l) {
        r.off_w[l] = L.off_w[l];
        r.off_b[l] = L.off_b[l];
        r.part_off[l] = L.part_off[l];
        r.out[l] = L.out[l];
        r.in[l] = L.in[l];
    }
    r.n_params = L.n_params;
    r.part_stride = L.part_stride;
    r.n_chunks = L.n_chunks;
    {
        ProfScope _r("k_mlp_reduce", s);
        hipLaunchKernelGGL(k_mlp_reduce, dim3((unsigned)((L.n_params + 255) / 256)), dim3(256), 0, s, r,
                           d.part, d_params);
        if (d_x0)
            hipLaunchKernelGGL(k_mlp_dx0, dim3((unsigned)((L.n + 255) / 256)), dim3(256), 0, s, dxr, L.n,
                               L.n_times, accumulate_x0 ? 1 : 0, d_x0);
    }
    return hipGetLastError();
}

hipError_t launch_decisions(const Layout& L, char* ws, uint8_t* dec, bool write, hipStream_t s) {
    if (!L.training) return hipErrorInvalidValue;
    uint4* mask = reinterpret_cast<uint4*>(ws + L.mask);
    const int64_t words = L.rows_pad / kRows * kDepth * 256;
    const unsigned blocks = (unsigned)((words + 255) / 256);
    if (write)
        hipLaunchKernelGGL(k_mlp_decisions<true>, dim3(blocks), dim3(256), 0, s, mask, dec, L.rows, words);
    else
        hipLaunchKernelGGL(k_mlp_decisions<false>, dim3(blocks), dim3(256), 0, s, mask, dec, L.rows, words);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace gft
