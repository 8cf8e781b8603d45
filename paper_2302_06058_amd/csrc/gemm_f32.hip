// fp32 N:M GEMM of Bi-Mask (Eq. 3 and Eq. 10 of arXiv 2302.06058) on gfx950:
//     C[t][a] = sum_k Bm[t][perm[k]] * A[a][k]        (perm = null: identity)
// with A in the fragment-major operand format of include/bimask.h, fp32 in, fp32 accumulation, fp32 out.
//
// fp32 layers are small (tens to hundreds of features and tokens), so what counts is the length of the chain of
// dependent memory round trips, not the rate: a workgroup owns one 16 x 16 output tile and its wavefronts split the
// CONTRACTION, 32 indices per wavefront and step, so that a layer of 128 inputs is one load round trip, 8 matrix
// instructions per wavefront and one reduction through LDS.  No operand passes through LDS: lane (c, q) = (l % 16,
// l / 16) of v_mfma_f32_16x16x4_f32 wants row c of either operand at contraction index q of four, and which four
// indices one instruction takes is free, so lane quarter q takes the 8 consecutive indices [8 q, 8 q + 8) of the step
// -- half a granule of the operand (16 bytes of slot values, 16 index bits) and 32 contiguous bytes of the token row.
// The column gather of Eq. (10) is in the token loads (4-byte loads through perm), not in a pass of its own.
// Products and sums are fp32 throughout; the wavefronts' partial sums are added in wavefront order.
//
// Measured (forward, W I x J at T tokens, 2:4): 64 x 128 at 32 22 -> 3.5 us (launch floor), 256 x 256 at 256 44 -> 3.7,
// 512 x 512 at 512 82 -> 9, 2048 x 2048 at 4096 956 -> 563 us, against one 64 x 64 tile of fmaf per workgroup that
// decoded the operand element by element into LDS; the error against float64 fell from 1.4e-7 .. 5.7e-7 to
// 0.8e-7 .. 2.9e-7 (shorter chains of additions).
#include "common.hpp"

namespace bimask {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 16;             // output tile: 16 weight rows x 16 tokens
constexpr int64_t kTilesX = 1 << 20;  // tiles in the x dimension of a launch at most

// one 8-index piece of a weight row: SPARSE: decoded from 4 slot values and 16 index bits
template <bool SPARSE>
struct WeightPiece {
    f32x4 v[SPARSE ? 1 : 2];
    uint32_t bits;
};

template <bool SPARSE>
__device__ __forceinline__ void load_weights(const float* __restrict__ A, const uint32_t* __restrict__ meta, int64_t row,
                                             int64_t k, int64_t ks, WeightPiece<SPARSE>& w) {
    if constexpr (SPARSE) {
        const int64_t g = k >> 2;                            // first of two groups: slots 2g .. 2g+3, nibbles g, g+1
        w.v[0] = *reinterpret_cast<const f32x4*>(A + tiled_val_off(row, 2 * g, ks));
        w.bits = meta[tiled_idx_word(row, g, ks)] >> (4 * (g & 7));
    } else {
        const float* p = A + tiled_dense_off(row, k, ks);
        w.v[0] = *reinterpret_cast<const f32x4*>(p);
        w.v[1] = *reinterpret_cast<const f32x4*>(p + 4);
    }
}

template <bool SPARSE>
__device__ __forceinline__ float weight_at(const WeightPiece<SPARSE>& w, int e) {      // e is compile-time after unrolling
    if constexpr (SPARSE) {
        const uint32_t nib = w.bits >> (4 * (e >> 2));
        const uint32_t p0 = nib & 3u, p1 = (nib >> 2) & 3u, pos = e & 3;
        const float hi = p1 == pos ? w.v[0][2 * (e >> 2) + 1] : 0.f;
        return p0 == pos ? w.v[0][2 * (e >> 2)] : hi;
    } else {
        return w.v[e >> 2][e & 3];
    }
}

template <bool SPARSE, bool PERM, int NW>
__global__ void __launch_bounds__(64 * NW)
k_gemm_f32(const float* __restrict__ A, const uint32_t* __restrict__ meta, int64_t Adim, int64_t K,
           const float* __restrict__ Bm, int64_t T, int64_t ldb, const int32_t* __restrict__ perm, float* __restrict__ C,
           int64_t ldc, uint32_t tiles_a, uint32_t tiles, bool vecB) {
    __shared__ float part[NW][4][64];
    const uint32_t tile = blockIdx.y * gridDim.x + blockIdx.x;
    if (tile >= tiles) return;                               // whole workgroup
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, q = lane >> 4;
    const uint32_t tt = tile / tiles_a;
    const int64_t a0 = static_cast<int64_t>(tile - tt * tiles_a) * kTile, t0 = static_cast<int64_t>(tt) * kTile;
    const int64_t ks = ceil_div(K, 128);
    const int64_t arow = a0 + c;                             // the operand is zero-padded to whole 32-row tiles
    const float* brow = Bm + (t0 + c < T ? t0 + c : T - 1) * ldb;      // clamped: computed, never stored

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t k0 = static_cast<int64_t>(wave) * 32; k0 < K; k0 += 32 * NW) {
        const int64_t k = k0 + 8 * q;                        // this lane's 8 contraction indices (weights zero beyond K)
        WeightPiece<SPARSE> w;
        load_weights<SPARSE>(A, meta, arow, k, ks, w);
        float b[8];
        if constexpr (PERM) {
            int col[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) col[e] = k + e < K ? perm[k + e] : -1;
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = col[e] >= 0 ? brow[col[e]] : 0.f;
        } else if (vecB) {                                   // K is a multiple of 4: whole 16-byte pieces
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                f32x4 x = {0.f, 0.f, 0.f, 0.f};
                if (k + 4 * v < K) x = *reinterpret_cast<const f32x4*>(brow + k + 4 * v);
#pragma unroll
                for (int e = 0; e < 4; ++e) b[4 * v + e] = x[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = k + e < K ? brow[k + e] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(weight_at<SPARSE>(w, e), b[e], acc, 0, 0, 0);
    }
    // lane (c, q) holds token c, weight rows 4 q .. 4 q + 3
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][r][lane] = acc[r];
    __syncthreads();
    if (tid < 256) {
        const int t = tid >> 4, a = tid & 15;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += part[w][a & 3][t + 16 * (a >> 2)];
        if (t0 + t < T && a0 + a < Adim) C[(t0 + t) * ldc + a0 + a] = s;
    }
}

template <bool SPARSE, bool PERM>
int run_f32(const float* A, const uint32_t* meta, int64_t Adim, int64_t K, const float* Bm, int64_t T, int64_t ldb,
            const int32_t* perm, float* C, int64_t ldc, hipStream_t s) {
    const int64_t tiles = ceil_div(T, kTile) * ceil_div(Adim, kTile);      // below 2^29: the output fits the card
    if (tiles > 0x7FFFFFFFll) return BIMASK_ERR_SHAPE;
    // A launch counts the work-items of a dimension in 32 bits and cuts off what is beyond, without an error: 2^24 tiles of
    // 256 threads in x alone would be none.  x holds 2^20 tiles (2^30 threads at most), y the rest.
    const uint32_t x = static_cast<uint32_t>(tiles < kTilesX ? tiles : kTilesX);
    const dim3 grid(x, static_cast<uint32_t>(ceil_div(tiles, x)));
    const bool vecB = aligned16(Bm) && ldb % 4 == 0;
#define BIMASK_GEMM_F32(NW)                                                                                   \
    hipLaunchKernelGGL((k_gemm_f32<SPARSE, PERM, NW>), grid, dim3(64 * NW), 0, s, A, meta, Adim, K, Bm, T, ldb, perm, C, ldc, \
                       static_cast<uint32_t>(ceil_div(Adim, kTile)), static_cast<uint32_t>(tiles), vecB)
    // few tiles: enough wavefronts that each has one or two steps; many tiles fill the chip by themselves
    if (tiles >= 2048 || K <= 128) BIMASK_GEMM_F32(4);
    else if (K <= 256) BIMASK_GEMM_F32(8);
    else BIMASK_GEMM_F32(16);
#undef BIMASK_GEMM_F32
    return check_launch();
}

}  // namespace

// The gather in the token loads costs one 4-byte load per token, contraction index and tile of 16 weight rows, the
// separate pass a launch and a read and write of the tokens.  256 x 256 at 256 tokens (64 Ki tile-indices): 4.6 us fused,
// 6.3 with the pass; 512 x 512 at 512 (512 Ki): 19 against 13.
bool gemm_f32_fuses_gather(int64_t T, int64_t Adim, int64_t K) {
    return ceil_div(T, kTile) * ceil_div(Adim, kTile) * K <= (1 << 17);
}

int launch_gemm_f32(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, bool sparse24, const void* Bm, int64_t T,
                    int64_t ldb, const int32_t* perm, void* C, int64_t ldc, hipStream_t s) {
    const float *a = static_cast<const float*>(A), *b = static_cast<const float*>(Bm);
    float* c = static_cast<float*>(C);
    if (sparse24) return perm ? run_f32<true, true>(a, meta, Adim, K, b, T, ldb, perm, c, ldc, s)
                              : run_f32<true, false>(a, meta, Adim, K, b, T, ldb, perm, c, ldc, s);
    return perm ? run_f32<false, true>(a, meta, Adim, K, b, T, ldb, perm, c, ldc, s)
                : run_f32<false, false>(a, meta, Adim, K, b, T, ldb, perm, c, ldc, s);
}

}  // namespace bimask
