// fp32 N:M GEMM of Bi-Mask (Eq. 3 and Eq. 10 of arXiv 2302.06058) on gfx950:
//     C[t][a] = sum_k Bm[t][perm[k]] * A[a][k]        (perm = null: identity)
// with A in the fragment-major operand format of include/bimask.h, fp32 in, fp32 accumulation, fp32 out.
//
// fp32 layers are small (tens to hundreds of features and tokens), so what counts is the length of the chain of
// dependent memory round trips, not the rate: a workgroup owns one 16 x 16 output tile (four of them side by side in large
// products) and its wavefronts split the CONTRACTION, 32 indices per wavefront and step, so that a layer of 128 inputs is one load round trip, 8 matrix
// instructions per wavefront and one reduction through LDS.  No operand passes through LDS: lane (c, q) = (l % 16,
// l / 16) of v_mfma_f32_16x16x4_f32 wants row c of either operand at contraction index q of four, and which four
// indices one instruction takes is free, so lane quarter q takes the 8 consecutive indices [8 q, 8 q + 8) of the step
// -- half a granule of the operand (16 bytes of slot values, 16 index bits) and 32 contiguous bytes of the token row.
// The column gather of Eq. (10) is in the token loads (4-byte loads through perm), not in a pass of its own.
// Products and sums are fp32 throughout; the wavefronts' partial sums are added in wavefront order.
//
// Measured (forward, W I x J at T tokens, 2:4): 64 x 128 at 32 22 -> 3.0 us (launch floor), 256 x 256 at 256 44 -> 3.2,
// 512 x 512 at 512 82 -> 8.3, 2048 x 2048 at 4096 957 -> 415, 512 x 8 at 401408 436 -> 284, against one 64 x 64 tile of fmaf
// per workgroup that decoded the operand element by element into LDS; the error against float64 fell from
// 1.4e-7 .. 5.7e-7 to 0.8e-7 .. 2.9e-7 (shorter chains of additions).
#include "common.hpp"

namespace bimask {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 16;             // output tile: 16 weight rows x 16 tokens
typedef f32x4 f32x4_row __attribute__((aligned(4)));      // 16 bytes of a token row: rows start on 4 bytes at least
constexpr int64_t kManyTiles = 8192;  // 16 x 16 tiles from which a workgroup takes 64 weight rows (one step: 4 times as many)
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

// R: row tiles of a workgroup (16 R weight rows x 16 tokens); the token pieces are loaded once for all of them and the output
// leaves in segments of 64 R bytes.  Token rows may start on any 4 bytes: the 16-byte loads need no more (256 x 256 at 50176
// tokens, rows of 1028 bytes, 4:8: 254 us with 4-byte loads, 85).
template <bool SPARSE, bool PERM, int NW, int R>
__global__ void __launch_bounds__(64 * NW)
k_gemm_f32(const float* __restrict__ A, const uint32_t* __restrict__ meta, int64_t Adim, int64_t K,
           const float* __restrict__ Bm, int64_t T, int64_t ldb, const int32_t* __restrict__ perm, float* __restrict__ C,
           int64_t ldc, uint32_t tiles_a, uint32_t tiles) {
    // partial sums [wave][row tile][register][lane]; strides that spread 64 consecutive outputs over all banks
    constexpr int SQ = 68, SR = 4 * SQ + 1;
    __shared__ float part[NW * R * SR];
    const uint32_t tile = blockIdx.y * gridDim.x + blockIdx.x;
    if (tile >= tiles) return;                               // whole workgroup
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, q = lane >> 4;
    const uint32_t tt = tile / tiles_a;
    const int64_t a0 = static_cast<int64_t>(tile - tt * tiles_a) * (kTile * R), t0 = static_cast<int64_t>(tt) * kTile;
    const int64_t ks = ceil_div(K, 128);
    const float* brow = Bm + (t0 + c < T ? t0 + c : T - 1) * ldb;      // clamped: computed, never stored

    f32x4 acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int64_t k0 = static_cast<int64_t>(wave) * 32; k0 < K; k0 += 32 * NW) {
        const int64_t k = k0 + 8 * q;                        // this lane's 8 contraction indices (weights zero beyond K)
        WeightPiece<SPARSE> w[R];
#pragma unroll
        for (int r = 0; r < R; ++r)                          // the operand is zero-padded to whole 32-row tiles, not further
            if (r == 0 || a0 + kTile * r < Adim) load_weights<SPARSE>(A, meta, a0 + kTile * r + c, k, ks, w[r]);
        float b[8];
        if constexpr (PERM) {
            int col[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) col[e] = k + e < K ? perm[k + e] : -1;
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = col[e] >= 0 ? brow[col[e]] : 0.f;
        } else {                                             // K is a multiple of 4: whole 16-byte pieces
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                f32x4 x = {0.f, 0.f, 0.f, 0.f};
                if (k + 4 * v < K) x = *reinterpret_cast<const f32x4_row*>(brow + k + 4 * v);
#pragma unroll
                for (int e = 0; e < 4; ++e) b[4 * v + e] = x[e];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r == 0 || a0 + kTile * r < Adim) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(weight_at<SPARSE>(w[r], e), b[e], acc[r], 0, 0, 0);
            }
    }
    // lane (c, q) holds token c, weight rows 4 q .. 4 q + 3 of every row tile
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[(wave * R + r) * SR + e * SQ + lane] = acc[r][e];
    __syncthreads();
    for (int i = tid; i < kTile * kTile * R; i += 64 * NW) {
        const int t = i / (kTile * R), a = i % (kTile * R);
        const float* p = part + (a >> 4) * SR + (a & 3) * SQ + t + 16 * ((a & 15) >> 2);
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += p[w * R * SR];
        if (t0 + t < T && a0 + a < Adim) C[(t0 + t) * ldc + a0 + a] = s;
    }
}

template <bool SPARSE, bool PERM, int NW, int R>
int run_f32_t(const float* A, const uint32_t* meta, int64_t Adim, int64_t K, const float* Bm, int64_t T, int64_t ldb,
              const int32_t* perm, float* C, int64_t ldc, hipStream_t s) {
    const int64_t tiles_a = ceil_div(Adim, kTile * R), tiles = ceil_div(T, kTile) * tiles_a;      // below 2^29: the output fits the card
    if (tiles > 0x7FFFFFFFll) return BIMASK_ERR_SHAPE;
    // A launch counts the work-items of a dimension in 32 bits and cuts off what is beyond, without an error: 2^24 tiles of
    // 256 threads in x alone would be none.  x holds 2^20 tiles (2^30 threads at most), y the rest.
    const uint32_t x = static_cast<uint32_t>(tiles < kTilesX ? tiles : kTilesX);
    const dim3 grid(x, static_cast<uint32_t>(ceil_div(tiles, x)));
    hipLaunchKernelGGL((k_gemm_f32<SPARSE, PERM, NW, R>), grid, dim3(64 * NW), 0, s, A, meta, Adim, K, Bm, T, ldb, perm, C, ldc,
                       static_cast<uint32_t>(tiles_a), static_cast<uint32_t>(tiles));
    return check_launch();
}

template <bool SPARSE, bool PERM>
int run_f32(const float* A, const uint32_t* meta, int64_t Adim, int64_t K, const float* Bm, int64_t T, int64_t ldb,
            const int32_t* perm, float* C, int64_t ldc, hipStream_t s) {
#define BIMASK_GEMM_F32(NW, R) return run_f32_t<SPARSE, PERM, NW, R>(A, meta, Adim, K, Bm, T, ldb, perm, C, ldc, s)
    const int64_t tiles = ceil_div(T, kTile) * ceil_div(Adim, kTile);
    // No wavefront without a step (512 x 8 at 401408 tokens: 812 us with 4 wavefronts of which 3 have nothing to do, 383 with
    // one).  Where 16 x 16 tiles fill the chip several times over, 64 weight rows per workgroup: fewer token loads and whole
    // lines out (the same 284 us; 2048 x 2048 at 4096 565 -> 415; 128 x 512 with 8192 tiles 41 -> 34, with 1024 8.7 / 9.4).
    // Up to 32 rows half of them would be idle (32 x 128 with 8192 tiles 15.1 / 16.0), and a single step gains from 32768
    // tiles on (128 x 16 with 8192 6.5 / 6.9, with 131072 51 -> 47).
    if constexpr (!PERM) {
        if (Adim > 2 * kTile && tiles >= (K <= 32 ? 4 * kManyTiles : kManyTiles)) {
            if (K <= 32) BIMASK_GEMM_F32(1, 4);
            if (K <= 64) BIMASK_GEMM_F32(2, 4);
            BIMASK_GEMM_F32(4, 4);
        }
    }
    if (K <= 32) BIMASK_GEMM_F32(1, 1);
    if (K <= 64) BIMASK_GEMM_F32(2, 1);
    // few tiles: enough wavefronts that each has one or two steps; many tiles fill the chip by themselves
    if (tiles >= 2048 || K <= 128) BIMASK_GEMM_F32(4, 1);
    if (K <= 256) BIMASK_GEMM_F32(8, 1);
    BIMASK_GEMM_F32(16, 1);
#undef BIMASK_GEMM_F32
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
