// N:M-sparse GEMMs of Bi-Mask (Eq. 3 and Eq. 10 of arXiv 2302.06058) on gfx950.
//
// Both directions are the same contraction   C[t][a] = sum_k Bm[t][k] * A[a][k]
//   forward : A = (B .* W)       (a = out feature i, k = in feature j),  Bm = X,      C = Y
//   backward: A = (Bbar.*W[P,:])^T (a = in feature j, k = permuted row r), Bm = dY[:,P], C = dX
// A is the weight operand: only the A side of a sparse matrix instruction may be 2:4
// compressed, so the weights sit on the A side and the product is formed transposed
// (rows of the accumulator tile are weight rows, columns are tokens).
//
// bf16, 2:4  : v_smfmac_f32_32x32x32_bf16 on the fragment-major compressed operand (gemm_sp24.hip)
// bf16, other: v_mfma_f32_32x32x16_bf16 on the dense masked weights (this file)
// fp32       : v_mfma_f32_16x16x4_f32, contraction split over the wavefronts (gemm_f32.hip)
#include "common.hpp"
#include <type_traits>

namespace bimask {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(__bf16)))) __bf16 bf16x16;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // native 16-byte register vector
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int BK = 64;                // dense k per pipeline stage
constexpr int kRowB = 144;            // LDS bytes per 64-k row (128 + 16 pad: conflict-free 16-byte reads)

// 8 consecutive bf16 of a row starting at element k (zero beyond kend).
__device__ __forceinline__ u32x4 load_granule(const uint16_t* row, int64_t k, int64_t kend, bool vec) {
    if (k + 8 <= kend) {
        if (vec) return *reinterpret_cast<const u32x4*>(row + k);
        const uint32_t* p = reinterpret_cast<const uint32_t*>(row + k);
        u32x4 r = {p[0], p[1], p[2], p[3]};
        return r;
    }
    u32x4 r = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (k + e < kend) r[e >> 1] |= static_cast<uint32_t>(row[k + e]) << (16 * (e & 1));
    return r;
}

template <int BM, int BN>
struct Smem {
    static constexpr int kA = BM * kRowB;
    static constexpr int kB = BN * kRowB;
    static constexpr int kStage = kA + kB;
    static constexpr int kCRow = BM * 2 + 16;
    static constexpr int kC = BN * kCRow;
    static constexpr int kTotal = (2 * kStage > kC) ? 2 * kStage : kC;
};

// Dense bf16 GEMM on masked weights (N:M ratios with N > 2), general fallback (any alignment, any
// contraction length).  Workgroup tile BM (weight rows a) x BN (tokens t); both operands go global ->
// registers -> padded LDS -> MFMA fragments, one stage prefetched in registers; the weight granules
// come from the fragment-major dense operand.
// FAST: K is a multiple of BK and all rows start 16-byte aligned: unconditional 16-byte loads.
template <bool FAST, int BM, int BN, int WAVES_M, int WAVES_N>
__global__ void __launch_bounds__(kThreads)
k_gemm_dense_bf16(const uint16_t* __restrict__ A, int64_t Adim, int64_t K, const uint16_t* __restrict__ Bm,
                  int64_t T, int64_t ldb, uint16_t* __restrict__ C, int64_t ldc, int tiles_a, bool vecA,
                  bool vecB, bool vecC) {
    static_assert(WAVES_M * WAVES_N == kThreads / 64, "four wavefronts");
    using S = Smem<BM, BN>;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    extern __shared__ u32x4 smem_u4[];
    uint8_t* smem = reinterpret_cast<uint8_t*>(smem_u4);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    const int l32 = lane & 31, h = lane >> 5;
    // Tile order as in the 2:4 kernel: workgroup ids are dealt round-robin to the 8 XCDs, so XCD x takes a
    // contiguous chunk of a sequence in which 8 token tiles x all weight tiles run side by side and share
    // that XCD's L2.
    constexpr int kGroupT = 8;
    const int64_t tiles_t = ceil_div(T, BN);
    const int64_t total = tiles_t * tiles_a;
    const int64_t per_xcd = ceil_div(total, 8);
    const int64_t n = static_cast<int64_t>(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (n >= total) return;
    const int64_t grp = n / (static_cast<int64_t>(kGroupT) * tiles_a);
    const int64_t first_t = grp * kGroupT;
    const int64_t gsz = (tiles_t - first_t) < kGroupT ? (tiles_t - first_t) : kGroupT;
    const int64_t within = n - grp * kGroupT * tiles_a;
    const int64_t a0 = (within / gsz) * BM;
    const int64_t t0 = (first_t + within % gsz) * BN;
    const int nk = static_cast<int>(ceil_div(K, BK));

    constexpr int NB_ = BN * 8 / kThreads, NA_ = BM * 8 / kThreads;   // 16-byte granules per thread
    u32x4 rb[NB_], ra[NA_];
    const uint16_t* pb[NB_];
    int64_t arow[NA_];                                   // weight row of each of this thread's granules (clamped)
#pragma unroll
    for (int it = 0; it < NB_; ++it) {
        int64_t t = t0 + ((tid + kThreads * it) >> 3);
        pb[it] = Bm + (t < T ? t : T - 1) * ldb;
    }
#pragma unroll
    for (int it = 0; it < NA_; ++it) {
        int64_t a = a0 + ((tid + kThreads * it) >> 3);
        arow[it] = a < Adim ? a : Adim - 1;
    }
    const int64_t ksA = ceil_div(K, 128);                // stages of the padded fragment-major weight operand
    const int g8 = (tid & 7) * 8;                        // this thread's k offset inside a stage

#define BIMASK_DENSE_LOAD(kt)                                                                     \
    {                                                                                             \
        const int64_t k = static_cast<int64_t>(kt) * BK + g8;                                     \
        _Pragma("unroll") for (int it = 0; it < NB_; ++it) {                                      \
            if constexpr (FAST) rb[it] = *reinterpret_cast<const u32x4*>(pb[it] + k);             \
            else rb[it] = load_granule(pb[it], k, K, vecB);                                       \
        }                                                                                         \
        /* the weight operand is padded to whole stages: every granule exists (zeros beyond K) */ \
        _Pragma("unroll") for (int it = 0; it < NA_; ++it)                                        \
            ra[it] = *reinterpret_cast<const u32x4*>(A + tiled_dense_off(arow[it], k, ksA));      \
    }
#define BIMASK_DENSE_STORE(buf)                                                                   \
    {                                                                                             \
        uint8_t* sA_ = smem + (buf) * S::kStage;                                                  \
        uint8_t* sB_ = sA_ + S::kA;                                                               \
        _Pragma("unroll") for (int it = 0; it < NB_; ++it)                                        \
            *reinterpret_cast<u32x4*>(sB_ + ((tid + kThreads * it) >> 3) * kRowB + (tid & 7) * 16) = rb[it]; \
        _Pragma("unroll") for (int it = 0; it < NA_; ++it)                                        \
            *reinterpret_cast<u32x4*>(sA_ + ((tid + kThreads * it) >> 3) * kRowB + (tid & 7) * 16) = ra[it]; \
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

    BIMASK_DENSE_LOAD(0)
    BIMASK_DENSE_STORE(0)
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const bool more = kt + 1 < nk;
        if (more) BIMASK_DENSE_LOAD(kt + 1)
        const uint8_t* sA = smem + (kt & 1) * S::kStage;
        const uint8_t* sB = sA + S::kA;
#pragma unroll
        for (int c = 0; c < 4; ++c) {                    // four 16-k MFMA steps per stage
            bf16x8 af[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[i] = *reinterpret_cast<const bf16x8*>(sA + (wm * WM + i * 32 + l32) * kRowB + c * 32 + h * 16);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const bf16x8 bf = *reinterpret_cast<const bf16x8*>(sB + (wn * WN + j * 32 + l32) * kRowB + c * 32 + h * 16);
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf, acc[i][j], 0, 0, 0);
            }
        }
        if (more) BIMASK_DENSE_STORE((kt + 1) & 1)
        __syncthreads();
    }
#undef BIMASK_DENSE_LOAD
#undef BIMASK_DENSE_STORE

    // Epilogue: accumulators -> bf16 tile [t][a] in LDS -> 16-byte row-contiguous stores.
    uint8_t* sC = smem;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int t = wn * WN + j * 32 + l32;
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                const int a = wm * WM + i * 32 + 8 * qq + 4 * h;
                u32x2 v;
                v.x = pack_bf16(acc[i][j][4 * qq + 0], acc[i][j][4 * qq + 1]);
                v.y = pack_bf16(acc[i][j][4 * qq + 2], acc[i][j][4 * qq + 3]);
                *reinterpret_cast<u32x2*>(sC + t * S::kCRow + a * 2) = v;
            }
        }
    __syncthreads();
    constexpr int GPR = BM / 8;                          // 16-byte granules per output row
    for (int q = tid; q < BN * GPR; q += kThreads) {
        const int row = q / GPR, g = q % GPR;
        const int64_t t = t0 + row, a = a0 + 8 * g;
        if (t >= T || a >= Adim) continue;
        const u32x4 v = *reinterpret_cast<const u32x4*>(sC + row * S::kCRow + g * 16);
        uint16_t* dst = C + t * ldc + a;
        if (vecC && a + 8 <= Adim) {
            *reinterpret_cast<u32x4*>(dst) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (a + e < Adim) dst[e] = static_cast<uint16_t>(v[e >> 1] >> (16 * (e & 1)));
        }
    }
}

// out[t][r] = in[t][perm[r]]   (the column permutation of g(Y) in Eq. 10)
template <typename raw>
__global__ void __launch_bounds__(kThreads)
k_gather_cols(const raw* __restrict__ in, int64_t T, int64_t ld, const int32_t* __restrict__ perm, int64_t I,
              raw* __restrict__ out, bool vec) {
    constexpr int E = 16 / sizeof(raw);
    const int64_t chunks = ceil_div(I, E);
    const int64_t id = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (id >= T * chunks) return;
    const int64_t t = id / chunks, r0 = (id - t * chunks) * E;
    const raw* src = in + t * ld;
    raw v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = (r0 + e < I) ? src[perm[r0 + e]] : static_cast<raw>(0);
    raw* dst = out + t * I + r0;
    if (vec && r0 + E <= I) {
        uint4 pk;
        if constexpr (sizeof(raw) == 2) {
            pk.x = v[0] | (static_cast<uint32_t>(v[1]) << 16); pk.y = v[2] | (static_cast<uint32_t>(v[3]) << 16);
            pk.z = v[4] | (static_cast<uint32_t>(v[5]) << 16); pk.w = v[6] | (static_cast<uint32_t>(v[7]) << 16);
        } else {
            pk.x = v[0]; pk.y = v[1]; pk.z = v[2]; pk.w = v[3];
        }
        *reinterpret_cast<uint4*>(dst) = pk;
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (r0 + e < I) dst[e] = v[e];
    }
}

// Same result, for rows that fit in LDS: a workgroup reads `rows` whole token rows with
// contiguous 16-byte lanes, keeps them in LDS, and every thread assembles 16-byte pieces of
// the permuted rows from 2- or 4-byte LDS reads.  Both global streams are fully coalesced.
// CPT > 0 (long rows): the grid is persistent, a thread owns the same CPT 16-byte output
// columns in every row tile and keeps their permutation entries in registers, so the
// permutation is read once per workgroup instead of once per row tile.
template <typename raw, int CPT>
__global__ void __launch_bounds__(kThreads)
k_gather_cols_lds(const raw* __restrict__ in, int64_t T, int64_t ld, const int32_t* __restrict__ perm, int64_t I,
                  raw* __restrict__ out, int rows, bool vec_in, bool vec_out) {
    constexpr int E = 16 / sizeof(raw);
    constexpr int NP = CPT > 0 ? CPT : 1;
    extern __shared__ uint4 gather_smem[];
    raw* buf = reinterpret_cast<raw*>(gather_smem);
    const int chunks = static_cast<int>(ceil_div(I, E));
    const int Ipad = chunks * E;
    const int64_t ntiles = ceil_div(T, rows);
    int p[NP][E];
    if constexpr (CPT > 0) {
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = threadIdx.x + kThreads * k;
#pragma unroll
            for (int e = 0; e < E; ++e) p[k][e] = (c * E + e < I) ? perm[c * E + e] : 0;
        }
    }
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t t0 = tile * rows;
        const int nrows = static_cast<int>((T - t0) < rows ? (T - t0) : rows);
        for (int idx = threadIdx.x; idx < nrows * chunks; idx += kThreads) {
            const int row = idx / chunks, c = idx - row * chunks;
            const raw* src = in + (t0 + row) * ld + static_cast<int64_t>(c) * E;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (vec_in && (c + 1) * E <= I) {
                v = *reinterpret_cast<const uint4*>(src);
            } else {
                uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (c * E + e < I) {
                        if constexpr (sizeof(raw) == 2) w[e >> 1] |= static_cast<uint32_t>(src[e]) << (16 * (e & 1));
                        else w[e] = src[e];
                    }
                v = make_uint4(w[0], w[1], w[2], w[3]);
            }
            *reinterpret_cast<uint4*>(buf + static_cast<int64_t>(row) * Ipad + c * E) = v;
        }
        __syncthreads();
        auto emit = [&](int c, const int (&pc)[E]) {
            for (int row = 0; row < nrows; ++row) {
                const raw* r = buf + static_cast<int64_t>(row) * Ipad;
                uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const uint32_t x = r[pc[e]];
                    if constexpr (sizeof(raw) == 2) w[e >> 1] |= x << (16 * (e & 1));
                    else w[e] = x;
                }
                raw* dst = out + (t0 + row) * I + static_cast<int64_t>(c) * E;
                if (vec_out && (c + 1) * E <= I) {
                    *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        if (c * E + e < I) {
                            if constexpr (sizeof(raw) == 2) dst[e] = static_cast<raw>(w[e >> 1] >> (16 * (e & 1)));
                            else dst[e] = w[e];
                        }
                }
            }
        };
        if constexpr (CPT > 0) {
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                const int c = threadIdx.x + kThreads * k;
                if (c < chunks) emit(c, p[k]);
            }
        } else {
            for (int c = threadIdx.x; c < chunks; c += kThreads) {
#pragma unroll
                for (int e = 0; e < E; ++e) p[0][e] = (c * E + e < I) ? perm[c * E + e] : 0;
                emit(c, p[0]);
            }
        }
        __syncthreads();                                 // the tile buffer is reused by the next row tile
    }
}

// The same gather for bf16 rows that are 16-byte aligned and a multiple of 8 long, with R = 2, 4 or 8 token rows
// per tile INTERLEAVED in LDS: element (column c, row r) sits at 2 (c R + r), so one LDS read of 2 R bytes at
// a permuted column returns that column for all R rows (R times fewer LDS reads than row-major tiles).  A
// thread owns the same CPT chunks of 8 columns in every tile, for the load (R global 16-byte loads per chunk,
// an 8 x R transpose of half-words in registers, R contiguous 16-byte LDS writes) and for the emit (8 LDS
// reads, the transpose back, R 16-byte stores), and keeps the chunks' permutation entries in registers as
// LDS byte offsets.  Persistent grid; the loads of the next tile are in flight while a tile is emitted.
// Bound by memory, with all of a tile's loads in flight at once: 22 KB rows (R = 2) at 8192 tokens 89 -> 71 us (5.1 TB/s; a plain
// device-to-device copy of the same arrays takes 64), the backward product with 8.5 KB rows (R = 4) at 9000 tokens 101 -> 91.
template <int R> struct GatherVec;
template <> struct GatherVec<2> { using type = uint32_t; };
template <> struct GatherVec<4> { using type = uint2; };
template <> struct GatherVec<8> { using type = uint4; };

template <int R, int CPT>
__global__ void __launch_bounds__(kThreads)
k_gather_cols_rows(const uint16_t* __restrict__ in, int64_t T, int64_t ld, const int32_t* __restrict__ perm, int I,
                   uint16_t* __restrict__ out) {
    using vec = typename GatherVec<R>::type;
    constexpr int W = R / 2;                             // dwords per column group
    extern __shared__ uint4 gather_smem[];
    uint8_t* buf = reinterpret_cast<uint8_t*>(gather_smem);
    const int chunks = I / 8;
    const int64_t ntiles = ceil_div(T, R);
    // Threads beyond the last chunk repeat it: no load or store but the last tile's is conditional.  (Behind a condition the
    // compiler cannot count what is in flight, and waits for the previous load and the previous tile's stores before each one:
    // 48 permutation entries and then 12 pieces a tile, one after the other.)
    int cc[CPT], p[CPT][8];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = threadIdx.x + kThreads * k;
        cc[k] = c < chunks ? c : chunks - 1;
#pragma unroll
        for (int e = 0; e < 8; ++e) p[k][e] = perm[cc[k] * 8 + e];
    }
    // the loads of a tile are issued before the previous tile is emitted: they are in flight during its LDS reads and stores
    uint4 v[CPT][R];
    auto load_tile = [&](int64_t tile) {
        const int64_t t0 = tile * R;
#pragma unroll
        for (int k = 0; k < CPT; ++k)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t t = t0 + r < T ? t0 + r : T - 1;          // rows beyond T repeat the last row (never stored)
                v[k][r] = *reinterpret_cast<const uint4*>(in + t * ld + cc[k] * 8);
            }
    };
    int64_t tile = blockIdx.x;                           // the grid is no larger than the number of tiles
    load_tile(tile);
#pragma unroll
    for (int k = 0; k < CPT; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) p[k][e] *= 2 * R;
    auto put_tile = [&]() {
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            // 8 columns x R rows: column e of the chunk -> R half-words (rows 0 .. R-1)
            uint32_t o[8][W];
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const uint32_t a = reinterpret_cast<const uint32_t*>(&v[k][2 * w])[e >> 1];
                    const uint32_t b = reinterpret_cast<const uint32_t*>(&v[k][2 * w + 1])[e >> 1];
                    o[e][w] = (e & 1) ? __builtin_amdgcn_perm(b, a, 0x07060302u) : __builtin_amdgcn_perm(b, a, 0x05040100u);
                }
            uint32_t* dst = reinterpret_cast<uint32_t*>(buf + static_cast<size_t>(cc[k]) * (16 * R));
#pragma unroll
            for (int q = 0; q < 8 * W; ++q)              // R 16-byte writes: 8 columns x W dwords
                if ((q & 3) == 0)
                    *reinterpret_cast<uint4*>(dst + q) = make_uint4(o[(q + 0) / W][(q + 0) % W], o[(q + 1) / W][(q + 1) % W],
                                                                    o[(q + 2) / W][(q + 2) % W], o[(q + 3) / W][(q + 3) % W]);
        }
    };
    auto emit_tile = [&](int64_t t0, auto last_c) {
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            uint32_t g[8][W];                            // permuted column e of the chunk, R rows
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const vec x = *reinterpret_cast<const vec*>(buf + p[k][e]);
#pragma unroll
                for (int w = 0; w < W; ++w) g[e][w] = reinterpret_cast<const uint32_t*>(&x)[w];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!decltype(last_c)::value || t0 + r < T) {
                    uint32_t wd[4];
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t a = g[2 * d][r >> 1], b = g[2 * d + 1][r >> 1];
                        wd[d] = (r & 1) ? __builtin_amdgcn_perm(b, a, 0x07060302u) : __builtin_amdgcn_perm(b, a, 0x05040100u);
                    }
                    typedef unsigned int gv4 __attribute__((ext_vector_type(4)));
                    const gv4 pk = {wd[0], wd[1], wd[2], wd[3]};
                    __builtin_nontemporal_store(pk, reinterpret_cast<gv4*>(out + (t0 + r) * I + cc[k] * 8));
                }
            }
        }
    };
    for (;;) {
        put_tile();
        __syncthreads();
        const int64_t next = tile + gridDim.x;
        if (next >= ntiles) break;
        load_tile(next);
        emit_tile(tile * R, std::false_type{});          // not the matrix's last tile: full
        tile = next;
        __syncthreads();                                 // the tile has been emitted
    }
    emit_tile(tile * R, std::true_type{});
}

// Columns of a fragment-major dense operand moved from permuted to natural order: out(r, P[k]) = in(r, k).  A dense
// operand has no structure along the contraction, so Eq. (10) is as well  dX = dY W'  with the columns of the weights put
// back where the columns of dY are, and the token matrix needs no gather.  Bound by its two passes over the operand:
// R rows of it per workgroup (R consecutive granules of 16 bytes in memory) meet in LDS, where the 2-byte scatter costs
// nothing next to the loads.  Backward product against a gathered copy of dY, 4:8: 384 x 1536 at 25216 tokens
// 56.7 -> 50.0 us, 2048 x 768 at 3000 35.4 -> 27.8, 1024 x 1024 at 8192 32.0 -> 25.6, 11008 x 4096 at 8192 733.7 -> 726.4.
__global__ void __launch_bounds__(kThreads)
k_unpermute_dense(const uint16_t* __restrict__ in, int K, int64_t ks, const int32_t* __restrict__ perm,
                  uint16_t* __restrict__ out, int log2r) {
    extern __shared__ uint4 unperm_smem[];
    uint16_t* lds = reinterpret_cast<uint16_t*>(unperm_smem);
    const int R = 1 << log2r, pitch = K + 8;             // K is a multiple of 8: LDS rows stay 16-byte aligned
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) << log2r;       // the operand is padded to whole 32-row tiles
    const int n = (K >> 3) << log2r, npad = static_cast<int>(ks * 16) << log2r;
    for (int c = threadIdx.x; c < n; c += kThreads) {
        const int r = c & (R - 1), k = (c >> log2r) * 8;
        const u32x4 v = *reinterpret_cast<const u32x4*>(in + tiled_dense_off(r0 + r, k, ks));
#pragma unroll
        for (int e = 0; e < 8; ++e) lds[r * pitch + perm[k + e]] = static_cast<uint16_t>(v[e >> 1] >> (16 * (e & 1)));
    }
    __syncthreads();
    for (int c = threadIdx.x; c < npad; c += kThreads) {
        const int r = c & (R - 1), k = (c >> log2r) * 8;
        u32x4 v = {0u, 0u, 0u, 0u};                      // padding of the contraction
        if (k < K) v = *reinterpret_cast<const u32x4*>(lds + r * pitch + k);
        *reinterpret_cast<u32x4*>(out + tiled_dense_off(r0 + r, k, ks)) = v;
    }
}

template <int R, int CPT>
int run_gather_rows(const void* dY, int64_t T, int64_t ld, const int32_t* perm, int64_t I, void* out, hipStream_t s) {
    auto kern = k_gather_cols_rows<R, CPT>;
    const size_t lds = static_cast<size_t>(I) * 2 * R;
    if (lds > 48 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess) return BIMASK_ERR_HIP;
    const int64_t ntiles = ceil_div(T, R);
    const int64_t per_cu = static_cast<int64_t>(160 * 1024 / lds) < 4 ? static_cast<int64_t>(160 * 1024 / lds) : 4;
    const unsigned grid = static_cast<unsigned>(ntiles < 256 * per_cu ? ntiles : 256 * per_cu);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, static_cast<const uint16_t*>(dY), T, ld, perm,
                       static_cast<int>(I), static_cast<uint16_t*>(out));
    return check_launch();
}

template <typename raw, int CPT>
int run_gather_lds(const void* dY, int64_t T, int64_t ld, const int32_t* perm, int64_t I, void* out, int rows,
                   size_t lds, unsigned grid, bool vec_in, bool vec_out, hipStream_t s) {
    auto kern = k_gather_cols_lds<raw, CPT>;
    if (lds > 48 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess) return BIMASK_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, static_cast<const raw*>(dY), T, ld, perm, I,
                       static_cast<raw*>(out), rows, vec_in, vec_out);
    return check_launch();
}

template <bool FAST, int BM, int BN, int WAVES_M, int WAVES_N>
int run_dense_t(const void* A, int64_t Adim, int64_t K, const void* Bm, int64_t T, int64_t ldb, void* C,
                int64_t ldc, hipStream_t s) {
    using S = Smem<BM, BN>;
    auto kern = k_gemm_dense_bf16<FAST, BM, BN, WAVES_M, WAVES_N>;
    if (S::kTotal > 48 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                S::kTotal) != hipSuccess) return BIMASK_ERR_HIP;
    }
    const bool vecA = aligned16(A) && (K * 2) % 16 == 0;
    const bool vecB = aligned16(Bm) && (ldb * 2) % 16 == 0;
    const bool vecC = aligned16(C) && (ldc * 2) % 16 == 0;
    const int tiles_a = static_cast<int>(ceil_div(Adim, BM));
    const int64_t tiles_t = ceil_div(T, BN);
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(ceil_div(tiles_a * tiles_t, 8) * 8)), dim3(kThreads), S::kTotal, s,
                       static_cast<const uint16_t*>(A), Adim, K, static_cast<const uint16_t*>(Bm), T, ldb,
                       static_cast<uint16_t*>(C), ldc, tiles_a, vecA, vecB, vecC);
    return check_launch();
}

int run_dense(const void* A, int64_t Adim, int64_t K, const void* Bm, int64_t T, int64_t ldb, void* C,
              int64_t ldc, hipStream_t s) {
    const bool fast = K % BK == 0 && aligned16(A) && aligned16(Bm) && (ldb * 2) % 16 == 0;
    if (fast) return run_dense_t<true, 128, 128, 2, 2>(A, Adim, K, Bm, T, ldb, C, ldc, s);
    return run_dense_t<false, 128, 128, 2, 2>(A, Adim, K, Bm, T, ldb, C, ldc, s);
}

}  // namespace

int launch_gather_cols(const void* dY, int64_t T, int64_t ld, const int32_t* perm, int64_t I, int dtype,
                       void* out, hipStream_t s) {
    const size_t esz = dtype == BIMASK_BF16 ? 2 : 4;
    const int64_t E = 16 / static_cast<int64_t>(esz);
    const size_t row_bytes = static_cast<size_t>(round_up(I, E)) * esz;
    if (row_bytes <= 64 * 1024) {
        // rows kept in LDS: as many as fit in 64 KB, but enough workgroups to fill the chip
        int64_t rows = static_cast<int64_t>((64 * 1024) / row_bytes);
        if (rows > 32) rows = 32;
        while (rows > 1 && ceil_div(T, rows) < 1024) rows /= 2;
        const size_t lds = static_cast<size_t>(rows) * row_bytes;
        const bool vec_in = aligned16(dY) && (ld * esz) % 16 == 0;
        const bool vec_out = aligned16(out) && (I * esz) % 16 == 0;
        const int64_t ntiles = ceil_div(T, rows);
        const int64_t cpt = ceil_div(ceil_div(I, E), kThreads);      // 16-byte output columns per thread
        // long aligned bf16 rows with enough of them: row-interleaved tiles.  Rows of 4-8 KB (2 chunks of 8 columns
        // per thread) fit 8 to a tile, of 8-16 KB (3-4 chunks) 4, of 16-24 KB (5-6 chunks) 2.
        if (dtype == BIMASK_BF16 && vec_in && vec_out && I % 8 == 0 && cpt >= 2 && cpt <= 6 && T >= 2048) {
            if (cpt <= 2) return run_gather_rows<8, 2>(dY, T, ld, perm, I, out, s);
            if (cpt <= 4) return run_gather_rows<4, 4>(dY, T, ld, perm, I, out, s);
            return run_gather_rows<2, 6>(dY, T, ld, perm, I, out, s);
        }
        // long rows: persistent grid (3 workgroups per CU), permutation entries in registers
        const bool persistent = cpt >= 2 && cpt <= 8;
        const unsigned grid = static_cast<unsigned>(persistent && ntiles > 768 ? 768 : ntiles);
        const int r = static_cast<int>(rows);
#define BIMASK_GATHER(RAW)                                                                                       \
        {                                                                                                        \
            if (!persistent) return run_gather_lds<RAW, 0>(dY, T, ld, perm, I, out, r, lds, grid, vec_in, vec_out, s); \
            if (cpt <= 2) return run_gather_lds<RAW, 2>(dY, T, ld, perm, I, out, r, lds, grid, vec_in, vec_out, s);    \
            if (cpt <= 4) return run_gather_lds<RAW, 4>(dY, T, ld, perm, I, out, r, lds, grid, vec_in, vec_out, s);    \
            if (cpt <= 6) return run_gather_lds<RAW, 6>(dY, T, ld, perm, I, out, r, lds, grid, vec_in, vec_out, s);    \
            return run_gather_lds<RAW, 8>(dY, T, ld, perm, I, out, r, lds, grid, vec_in, vec_out, s);                  \
        }
        if (dtype == BIMASK_BF16) BIMASK_GATHER(uint16_t)
        BIMASK_GATHER(uint32_t)
#undef BIMASK_GATHER
    }
    if (dtype == BIMASK_BF16) {
        const int64_t total = T * ceil_div(I, 8);
        const bool vec = aligned16(out) && (I * 2) % 16 == 0;
        hipLaunchKernelGGL(k_gather_cols<uint16_t>, dim3(static_cast<unsigned>(ceil_div(total, kThreads))),
                           dim3(kThreads), 0, s, static_cast<const uint16_t*>(dY), T, ld, perm, I,
                           static_cast<uint16_t*>(out), vec);
    } else {
        const int64_t total = T * ceil_div(I, 4);
        const bool vec = aligned16(out) && (I * 4) % 16 == 0;
        hipLaunchKernelGGL(k_gather_cols<uint32_t>, dim3(static_cast<unsigned>(ceil_div(total, kThreads))),
                           dim3(kThreads), 0, s, static_cast<const uint32_t*>(dY), T, ld, perm, I,
                           static_cast<uint32_t*>(out), vec);
    }
    return check_launch();
}

namespace {
constexpr int64_t kUnpermuteLds = 48 * 1024;             // one row of the operand has to fit
// operand rows per workgroup (log2): 8 = whole 128-byte lines; fewer for long rows or few rows
int unpermute_rows_log2(int64_t I, int64_t rows) {
    int log2r = 3;
    while (log2r > 0 && ((I + 8) * 2 << log2r) > kUnpermuteLds) --log2r;
    while (log2r > 2 && (rows >> log2r) < 512) --log2r;
    return log2r;
}
}  // namespace

// Weight bytes (padded) up to those of the tokens: both passes read and write what they move once.  Where LDS takes only two
// rows or one, the operand moves as 32- or 16-byte pieces and the line is lower: 8192 x 2240 at 3000 tokens 137 us with the
// gathered copy, 144 un-permuted, 8192 x 2048 134 / 134; 16384 x 1472 at 3000 283 / 313, 16384 x 1024 210 / 210.  The product
// then reads dY itself, so its rows have to be 16-byte aligned.
bool gemm_dense_unpermutes(const void* dY, int64_t T, int64_t ld, int64_t J, int64_t I) {
    if (I % 8 != 0 || (I + 8) * 2 > kUnpermuteLds || !aligned16(dY) || ld % 8 != 0) return false;
    const int64_t weights = round_up(J, 32) * round_up(I, 128), tokens = T * I;
    const int log2r = unpermute_rows_log2(I, round_up(J, 32));
    return log2r >= 2 ? weights <= tokens : log2r == 1 ? 3 * weights <= 2 * tokens : 3 * weights <= tokens;
}

int launch_unpermute_dense(const void* values, int64_t J, int64_t I, const int32_t* perm, void* out, hipStream_t s) {
    const int64_t rows = round_up(J, 32);
    const int log2r = unpermute_rows_log2(I, rows);
    const size_t lds = static_cast<size_t>((I + 8) * 2) << log2r;
    hipLaunchKernelGGL(k_unpermute_dense, dim3(static_cast<unsigned>(rows >> log2r)), dim3(kThreads), lds, s,
                       static_cast<const uint16_t*>(values), static_cast<int>(I), ceil_div(I, 128), perm,
                       static_cast<uint16_t*>(out), log2r);
    return check_launch();
}

bool gemm_bwd_needs_gather(int64_t I, int64_t J, int dtype, int N, int M) {
    if (dtype != BIMASK_BF16) return true;
    if (!uses_sp24(N, M)) return !gemm_dense_coltile_shape(J, I);
    return !(I <= 512 || gemm_sp24_coltile_shape(J, I));
}

int launch_gemm(const void* A_values, const uint32_t* A_index, int64_t Adim, int64_t K, bool sparse24,
                const void* Bm, int64_t T, int64_t ldb, void* C, int64_t ldc, int dtype, hipStream_t s) {
    if (dtype == BIMASK_F32) return launch_gemm_f32(A_values, A_index, Adim, K, sparse24, Bm, T, ldb, nullptr, C, ldc, s);
    const int rc = launch_gemm_sp24_wide(A_values, A_index, Adim, K, Bm, ldb, nullptr, T, C, ldc, s, !sparse24);
    if (rc != BIMASK_ERR_UNSUPPORTED) return rc;
    if (sparse24) {
        // A 64 x 32 or 64 x 64 tile per CU at most: split the contraction inside the workgroup (4096 x 4096 at 64 tokens
        // 17.5 -> 8.9 us, at 256 18.3 -> 15.4).  Three stages and more gain, four where token rows are read in 4-byte pieces
        // (512 x 264 at 64 tokens 4.6 -> 4.1 us; 512 x 260 with rows of 524 bytes 6.0, split 6.6).  One stage has nothing to
        // split; two pay for it only against the resident kernel, with 16-byte token rows and enough of them (512 x 192 at 64
        // tokens 5.1 -> 4.0 us, at 4 tokens 3.8 / 3.9; 512 x 256, streamed otherwise, at 16 3.8 / 4.1; 4-byte pieces
        // 512 x 132 at 32 5.2 / 6.4).  Up to 64 rows the 64 x 64 tile is the shorter with one group (64 x 576 at 13000 tokens
        // 5.1 us, two groups 5.9).
        const bool rows16 = aligned16(Bm) && ldb % 8 == 0 && K % 8 == 0, deep = K > (rows16 ? 256 : 384);
        const bool two_stages = rows16 && K > 128 && T >= 16 && (K < 256 || Adim > 512);
        const bool split32 = (deep || two_stages) && gemm_few_tiles(Adim, T);
        const bool split64 = deep && Adim > 64 && ceil_div(Adim, 64) * ceil_div(T, 64) <= 256;
        if (K <= 512) {
            // narrow weights: wavefront-private tiles; short contractions (below 256, or below 384 with more
            // than 512 weight rows): token tile resident in LDS, reused by every weight tile; otherwise the
            // streaming kernel below (measured per layer shape: 128 x 512 forward 30 -> 20 us, 2048 x 512 14 -> 10 us)
            int rc = launch_gemm_sp24_narrow(A_values, A_index, Adim, K, Bm, ldb, nullptr, T, C, ldc, s);
            if (rc != BIMASK_ERR_UNSUPPORTED) return rc;
            // (with few tokens a workgroup or two would walk all weight rows: 2048 x 256 at 64 tokens 5.3 us resident, 4.4 split)
            if ((K < 256 || (K < 384 && Adim > 512)) && !split32) {
                rc = launch_gemm_sp24_resident(A_values, A_index, Adim, K, Bm, ldb, nullptr, T, C, ldc, s);
                if (rc != BIMASK_ERR_UNSUPPORTED) return rc;
            }
        }
        // the largest problems: 512 x 128 tiles, wavefronts of 64 x 128 (fewest L2 and LDS bytes per matrix instruction)
        if (gemm_sp24_big_shape(Adim, K, T)) {
            const int rc = launch_gemm_sp24_big(A_values, A_index, Adim, K, Bm, T, ldb, C, ldc, s);
            if (rc != BIMASK_ERR_UNSUPPORTED) return rc;
        }
        // large problems: 256 x 128 tiles on 8 wavefronts (half the weight traffic per token);
        // otherwise 256 x 64 tiles so that the grid still covers the chip; weight dimensions that
        // would leave a fifth or more of the 256-row tiles empty (384 = 1.5 tiles) take 128-row tiles
        const bool big = ceil_div(Adim, 256) * ceil_div(T, 128) >= 190;
        const int64_t w256 = round_up(Adim, 256), w128 = round_up(Adim, 128);
        const bool narrow = (w256 - w128) * 5 >= w256;
        // few tokens and few weight tiles: 256-row tiles would leave CUs idle
        const bool underfilled = ceil_div(Adim, 256) * ceil_div(T, 64) <= 128;
        const Sp24Tile tile = split32 ? Sp24Tile::k64x32Split
                            : split64 ? Sp24Tile::k64x64Split
                            : Adim <= 64 ? Sp24Tile::k64x64
                            : narrow || underfilled ? Sp24Tile::k128x64
                            : big ? Sp24Tile::k256x128 : Sp24Tile::k256x64;
        return launch_gemm_sp24(A_values, A_index, Adim, K, Bm, T, ldb, C, ldc, tile, s);
    }
    {   // dense masked weights: the streaming kernel on the fragment-major operand; else the general kernel
        const int rc = launch_gemm_dense_frag(A_values, Adim, K, Bm, T, ldb, C, ldc, s);
        if (rc != BIMASK_ERR_UNSUPPORTED) return rc;
    }
    return run_dense(A_values, Adim, K, Bm, T, ldb, C, ldc, s);
}

}  // namespace bimask
