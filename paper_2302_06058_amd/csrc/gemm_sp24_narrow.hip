// 2:4-sparse bf16 GEMM for narrow weights and short contractions, wavefront-private variant:
//     C[t][a] = sum_k Bsrc[t][perm[k]] * A[a][k],   a < Adim <= 256,  k < K <= 512
// (Eq. (3) / Eq. (10) of arXiv 2302.06058 for layers with few features on both sides of the
// weight matrix: the first convolutions of a ResNet, whose token count is in the hundreds of
// thousands.)  Such a layer is a pure stream: ~300 bytes in and ~130 bytes out per token and
// a handful of matrix instructions, so what matters is the instruction count per token.
//
// One wavefront owns one tile of 32 tokens at a time and shares nothing with other
// wavefronts: the compressed weights of ALL weight rows live in its registers for the whole
// kernel, the token rows travel global -> registers -> LDS as whole 16-byte pieces (requested
// one tile ahead), every token fragment is read from LDS exactly once, and the 32 x Adim
// output tile is regrouped through the same LDS area into whole rows that leave with
// streaming stores.  No workgroup barrier anywhere; LDS rows sit at a pitch whose dword
// stride is 2 x odd, which makes the 8-byte accesses of 32 lanes (one per token) hit 64
// distinct banks.  Rows whose byte length is no multiple of 16 (K or Adim = 8 m + 4) must be
// contiguous in memory; a 32-token tile is then one 16-byte-aligned block.
#include "common.hpp"
#include <type_traits>

namespace bimask {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(__bf16)))) __bf16 bf16x16;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

union BFragN { bf16x16 v; u32x4 q[2]; };
union AFragN { bf16x8 v; u32x4 q; };

__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// LDS pitch of a row of `w` bf16: the row itself, plus 8 bytes when that is a multiple of 16
__host__ __device__ inline int narrow_pitch(int w) { return (w & 7) ? 2 * w : 2 * w + 8; }

// registers: TM * NSTG * 18 for the weights, TM * 16 accumulators, NSTG * 32 for the rows in flight;
// two wavefronts per SIMD (256 registers each) except for the longest contractions
constexpr int narrow_waves_per_simd(int tm, int nstg) { return nstg >= 4 || (nstg == 3 && tm >= 2) ? 1 : 2; }

template <int TM, int NSTG>
__global__ void __launch_bounds__(64, narrow_waves_per_simd(TM, NSTG))
k_gemm_sp24_narrow(const uint16_t* __restrict__ A_all, const uint32_t* __restrict__ Ameta_all, int Adim_all, int K,
                   const uint16_t* __restrict__ Bsrc, int ldb, const int32_t* __restrict__ perm, int64_t T,
                   uint16_t* __restrict__ C_all, int ldc, int nsplit, bool stream_out) {
    // Weight rows beyond TM * 32 are split over `nsplit` wavefronts that work on the same token
    // tile; workgroups 8 apart run on the same XCD, so the tile is fetched from memory once.
    const int split = (static_cast<int>(blockIdx.x) >> 3) % nsplit;
    const int64_t wave_id = ((static_cast<int64_t>(blockIdx.x) >> 3) / nsplit) * 8 + (blockIdx.x & 7);
    const int64_t nwaves = gridDim.x / nsplit;
    // row tiles of this split; the last split may own fewer than TM (7 row tiles over 2 x 4): its
    // surplus tiles re-read the operand's last row tile (loaded, never stored)
    const int rt_last = (Adim_all + 31) / 32 - 1;
    uint16_t* __restrict__ C = C_all + split * TM * 32;
    const int Adim = Adim_all - split * TM * 32 < TM * 32 ? Adim_all - split * TM * 32 : TM * 32;
    // q / G == (q * invG) >> 22 for q < 64, G <= 64
    const int invG_arg = (K & 7) ? 0 : ((1 << 22) + (K >> 3) - 1) / (K >> 3);
    const int invU_arg = (Adim & 7) ? 0 : ((1 << 22) + (Adim >> 3) - 1) / (Adim >> 3);
    const int dtB = (K & 7) ? 0 : 64 / (K >> 3), dgB = (K & 7) ? 0 : 64 % (K >> 3);
    const int dtC = (Adim & 7) ? 0 : 64 / (Adim >> 3), dgC = (Adim & 7) ? 0 : 64 % (Adim >> 3);
    extern __shared__ u32x4 smem_u4[];
    uint8_t* smem = reinterpret_cast<uint8_t*>(smem_u4);
    int32_t* sInv = reinterpret_cast<int32_t*>(smem);        // byte offset of column c inside a permuted row
    uint8_t* area = smem + NSTG * 512;                       // token rows, later the output rows

    // Everything below that depends only on the lane or on the shape is the same for every tile.
    // The values are re-derived per tile from copies the optimiser cannot see through: hoisted
    // out of the tile loop they would occupy a few hundred registers for the whole kernel.
#define BIMASK_NARROW_SHAPE(LANE_SRC, K_SRC, A_SRC)                                              \
    int lane = (LANE_SRC), Kq = (K_SRC), Aq = (A_SRC);                                           \
    asm volatile("" : "+v"(lane));                                                               \
    asm volatile("" : "+s"(Kq));                                                                 \
    asm volatile("" : "+s"(Aq));                                                                 \
    const int l32 = lane & 31, h = lane >> 5;                                                    \
    const bool packB = (Kq & 7) != 0, packC = (Aq & 7) != 0;                                     \
    const int pitchB = narrow_pitch(Kq), pitchC = narrow_pitch(Aq);                              \
    const int G = Kq >> 3, UPR = Aq >> 3;            /* 16-byte pieces per row (aligned rows) */ \
    /* 16-byte piece q = lane + 64 it of a tile is piece g of row t with q = t G + g; the walk from \
       one `it` to the next adds 64 = dt G + dg and carries when g passes G (no divisions) */    \
    const int tB0 = static_cast<int>(static_cast<uint32_t>(lane * invG_arg) >> 22), gB0 = lane - tB0 * G; \
    const int tC0 = static_cast<int>(static_cast<uint32_t>(lane * invU_arg) >> 22), gC0 = lane - tC0 * UPR; \
    const bool Kfull = Kq == NSTG * 128;                                                         \
    const bool Afull = Aq == TM * 32;                                                            \
    (void)l32; (void)h; (void)packC; (void)pitchC; (void)UPR; (void)Kfull; (void)Afull; (void)pitchB; (void)G; (void)packB; (void)tB0; (void)gB0; (void)tC0; (void)gC0;
    const int lane0 = threadIdx.x;
    constexpr int NLD = NSTG * 8;                            // 16-byte pieces of 32 token rows per lane, at most
    constexpr int NOUT = TM * 2;                             // the same for the output rows

    const int64_t ntiles = ceil_div(T, 32);
    int64_t tile = wave_id;
    if (tile >= ntiles) return;

    // ---- all weight fragments: NSTG stages x TM row tiles x 4 sub-steps, for the whole kernel
    u32x4 ra[NSTG][TM][4];
    u32x2 rmeta[NSTG][TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int rt = split * TM + i < rt_last ? split * TM + i : rt_last;
        const uint16_t* pa = A_all + (static_cast<int64_t>(rt) * NSTG * 256 + lane0) * 8;
        const uint32_t* pm = Ameta_all + (static_cast<int64_t>(rt) * NSTG * 64 + lane0) * 2;
#pragma unroll
        for (int st = 0; st < NSTG; ++st) {
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4)
                ra[st][i][s4] = *reinterpret_cast<const u32x4*>(pa + (st * 4 + s4) * 512);
            rmeta[st][i] = *reinterpret_cast<const u32x2*>(pm + st * 128);
        }
    }

    // ---- token rows of one tile -> registers
    u32x4 v[NLD];
#define BIMASK_NARROW_LOAD(TILE)                                                                 \
    {                                                                                            \
        const int64_t t0_ = (TILE) * 32;                                                         \
        const int rows_ = static_cast<int>((T - t0_) < 32 ? (T - t0_) : 32);                     \
        if (packB) {                                                                             \
            const int nbytes = rows_ * Kq * 2;                                                    \
            const uint16_t* blk = Bsrc + t0_ * Kq;                                                \
            _Pragma("unroll") for (int it = 0; it < NLD; ++it) {                                 \
                const int q = lane + 64 * it;                                                    \
                v[it] = (u32x4){0u, 0u, 0u, 0u};                                                 \
                if (it * 1024 < nbytes) {                                                        \
                    if (q * 16 + 16 <= nbytes) v[it] = reinterpret_cast<const u32x4*>(blk)[q];   \
                    else if (q * 16 < nbytes) {      /* odd row count: the block ends in 8 bytes */ \
                        const u32x2 t2 = *reinterpret_cast<const u32x2*>(blk + q * 8);           \
                        v[it].x = t2.x; v[it].y = t2.y;                                          \
                    }                                                                            \
                }                                                                                \
            }                                                                                    \
        } else {                                                                                 \
            const uint16_t* base = Bsrc + t0_ * ldb;                                             \
            const int step = dtB * ldb + 8 * dgB, carry = ldb - 8 * G, end = rows_ * ldb;        \
            int g = gB0, ofs = tB0 * ldb + 8 * gB0;          /* element offset of the piece */   \
            _Pragma("unroll") for (int it = 0; it < NLD; ++it) {                                 \
                v[it] = (u32x4){0u, 0u, 0u, 0u};                                                 \
                if (it * 64 < 32 * G) {                                                          \
                    if (ofs < end) v[it] = *reinterpret_cast<const u32x4*>(base + ofs);          \
                    g += dgB; ofs += step;                                                       \
                    if (g >= G) { g -= G; ofs += carry; }                                        \
                }                                                                                \
            }                                                                                    \
        }                                                                                        \
    }
    {
        BIMASK_NARROW_SHAPE(lane0, K, Adim)
        BIMASK_NARROW_LOAD(tile)
    }

    if (perm) {             // Eq. (10) reads column P[k] at position k: column c = P[k] is stored at 2 k
        for (int r = lane0; r < K; r += 64) sInv[perm[r]] = 2 * r;
    }

    for (;;) {
        BIMASK_NARROW_SHAPE(lane0, K, Adim)
        const int64_t t0 = tile * 32;
        const int rows = static_cast<int>((T - t0) < 32 ? (T - t0) : 32);
        wave_lds_fence();                                    // the previous tile's output rows have been read
        // ---- registers -> LDS rows (rows beyond `rows` are zeros)
        if (packB) {
#pragma unroll
            for (int it = 0; it < NLD; ++it) {
                const int q = lane + 64 * it;
                if (it * 1024 < 32 * pitchB && q * 16 < 32 * pitchB) *reinterpret_cast<u32x4*>(area + q * 16) = v[it];
            }
        } else if (perm) {
            // the column gather of Eq. (10), done as a scatter on the way into LDS: 2-byte stores
            const int step = dtB * pitchB, end = 32 * pitchB;
            int g = gB0, rofs = tB0 * pitchB;                // byte offset of the piece's row
#pragma unroll
            for (int it = 0; it < NLD; ++it) {
                if (it * 64 < 32 * G) {
                    if (rofs < end) {
                        const u32x4 i0 = *reinterpret_cast<const u32x4*>(sInv + 8 * g);
                        const u32x4 i1 = *reinterpret_cast<const u32x4*>(sInv + 8 * g + 4);
                        uint8_t* row = area + rofs;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const uint32_t off = e < 4 ? i0[e] : i1[e - 4];
                            *reinterpret_cast<uint16_t*>(row + off) = static_cast<uint16_t>(v[it][e >> 1] >> (16 * (e & 1)));
                        }
                    }
                    g += dgB; rofs += step;
                    if (g >= G) { g -= G; rofs += pitchB; }
                }
            }
        } else {
            const int step = dtB * pitchB + 16 * dgB, carry = pitchB - 16 * G, end = 32 * pitchB;
            int g = gB0, ofs = tB0 * pitchB + 16 * gB0;      // byte offset of the piece in LDS
#pragma unroll
            for (int it = 0; it < NLD; ++it) {
                if (it * 64 < 32 * G) {
                    if (ofs < end) {
                        u32x2* d = reinterpret_cast<u32x2*>(area + ofs);
                        d[0] = (u32x2){v[it].x, v[it].y};
                        d[1] = (u32x2){v[it].z, v[it].w};
                    }
                    g += dgB; ofs += step;
                    if (g >= G) { g -= G; ofs += carry; }
                }
            }
        }
        wave_lds_fence();
        const int64_t next = tile + nwaves;
        if (next < ntiles) BIMASK_NARROW_LOAD(next)          // in flight during this tile's arithmetic

        // ---- NSTG x 4 sparse matrix instructions per weight-row tile
        f32x16 acc[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][q] = 0.f;
        const uint8_t* myrow = area + l32 * pitchB;
#pragma unroll
        for (int st = 0; st < NSTG; ++st) {
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                BFragN bf;
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const int k0 = 8 * (st * 16 + 8 * x + 2 * s4 + h);      // this lane's 8 contraction indices
                    const u32x2* p = reinterpret_cast<const u32x2*>(myrow + 2 * k0);
                    const u32x2 lo = p[0], hi = p[1];
                    u32x4 o = {lo.x, lo.y, hi.x, hi.y};
                    if (!Kfull) {                            // beyond K: whatever LDS holds there
#pragma unroll
                        for (int d = 0; d < 4; ++d)
                            if (k0 + 2 * d + 2 > Kq) o[d] = 0u;
                    }
                    bf.q[x] = o;
                }
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    AFragN af;
                    af.q = ra[st][i][s4];
                    const int idx = static_cast<int>(s4 < 2 ? rmeta[st][i].x : rmeta[st][i].y);
                    if (s4 & 1)
                        acc[i] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, bf.v, acc[i], idx, 0, 1);
                    else
                        acc[i] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, bf.v, acc[i], idx, 0, 0);
                }
            }
        }

        // ---- output.  A lane holds 4 consecutive weight rows of its token per accumulator quad;
        // swapping quads between the lane halves gives it 8 consecutive bf16 (16 bytes) of the
        // token's output row, which go to LDS at the output pitch.
        wave_lds_fence();                                    // all fragment reads precede the overwrite
        uint8_t* orow = area + l32 * pitchC;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const uint32_t xlo = pack_bf16(acc[i][8 * p + 0], acc[i][8 * p + 1]);
                const uint32_t xhi = pack_bf16(acc[i][8 * p + 2], acc[i][8 * p + 3]);
                const uint32_t ylo = pack_bf16(acc[i][8 * p + 4], acc[i][8 * p + 5]);
                const uint32_t yhi = pack_bf16(acc[i][8 * p + 6], acc[i][8 * p + 7]);
                const auto slo = __builtin_amdgcn_permlane32_swap(xlo, ylo, false, false);
                const auto shi = __builtin_amdgcn_permlane32_swap(xhi, yhi, false, false);
                const int a0 = i * 32 + 16 * p + 8 * h;      // first of this lane's 8 weight rows
                if (Afull || a0 + 8 <= Aq) {
                    u32x2* d = reinterpret_cast<u32x2*>(orow + 2 * a0);
                    d[0] = (u32x2){slo[0], shi[0]};
                    d[1] = (u32x2){slo[1], shi[1]};
                } else {
                    uint32_t* d = reinterpret_cast<uint32_t*>(orow + 2 * a0);
                    if (a0 + 2 <= Aq) d[0] = slo[0];
                    if (a0 + 4 <= Aq) d[1] = shi[0];
                    if (a0 + 6 <= Aq) d[2] = slo[1];
                }
            }
        wave_lds_fence();
        if (packC) {                                         // the tile is one aligned block of the output
            const int nbytes = rows * Aq * 2;
            uint16_t* blk = C + t0 * Aq;
#pragma unroll
            for (int it = 0; it < NOUT; ++it) {
                const int q = lane + 64 * it;
                if (it * 1024 < nbytes) {
                    if (q * 16 + 16 <= nbytes) {
                        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(area + q * 16), reinterpret_cast<u32x4*>(blk) + q);
                    } else if (q * 16 < nbytes) {            // odd row count: the block ends in 8 bytes
                        *reinterpret_cast<u32x2*>(blk + q * 8) = *reinterpret_cast<const u32x2*>(area + q * 16);
                    }
                }
            }
        } else {
            uint16_t* base = C + t0 * ldc;
            const int lstep = dtC * pitchC + 16 * dgC, lcarry = pitchC - 16 * UPR;
            const int gstep = dtC * ldc + 8 * dgC, gcarry = ldc - 8 * UPR, end = rows * ldc;
            int u = gC0, lofs = tC0 * pitchC + 16 * gC0, gofs = tC0 * ldc + 8 * gC0;
#pragma unroll
            for (int it = 0; it < NOUT; ++it) {
                if (it * 64 < 32 * UPR) {
                    if (gofs < end) {
                        const u32x2* p = reinterpret_cast<const u32x2*>(area + lofs);
                        const u32x2 lo = p[0], hi = p[1];
                        const u32x4 o = {lo.x, lo.y, hi.x, hi.y};
                        u32x4* dst = reinterpret_cast<u32x4*>(base + gofs);
                        store16(o, dst, stream_out);
                    }
                    u += dgC; lofs += lstep; gofs += gstep;
                    if (u >= UPR) { u -= UPR; lofs += lcarry; gofs += gcarry; }
                }
            }
        }
        if (next >= ntiles) break;
        tile = next;
    }
#undef BIMASK_NARROW_LOAD
#undef BIMASK_NARROW_SHAPE
}

// Rows that are no multiple of 16 bytes stay with the kernel above, and a few gathers (gemm_sp24_narrow_streams).
// Token rows and output rows in 16-byte pieces (K and Adim multiples of 8): every load and every store of a tile is unconditional,
// which is what keeps the next tile's rows in flight.  Where a piece is loaded under a condition the compiler cannot count what is
// outstanding and waits for the previous load -- and for the previous tile's stores -- before each one.  Pieces and rows that do
// not exist repeat one that does (loads), go to a spare row (LDS) or store the last piece once more; all tiles but the last one of
// the matrix are full, and only that one's stores are conditional.  Bound by memory; the kernel above, with conditions -> this
// one, us (means over four cards, buffers in turn): 64 -> 256 columns at 200704 tokens 34.5 -> 23.3 (5.5 TB/s), with the gather
// 36.9 -> 23.8, 128 -> 256 with the gather 41.0 -> 28.4, 512 -> 64 at 100000 38.2 -> 28.1, 64 -> 128 at 3000 5.0 -> 3.0.
// NP: pieces per lane and tile (K <= 16 NP); WHOLE: K = 16 NP and Adim a multiple of 32 TM, known at compile time.
template <int TM, int NP, bool PERM, bool WHOLE>
__global__ void __launch_bounds__(64, narrow_waves_per_simd(TM, (NP + 7) / 8))
k_gemm_sp24_narrow_rows(const uint16_t* __restrict__ A_all, const uint32_t* __restrict__ Ameta_all, int Adim_all, int K_arg,
                        const uint16_t* __restrict__ Bsrc, int ldb, const int32_t* __restrict__ perm, int64_t T,
                        uint16_t* __restrict__ C_all, int ldc, int nsplit, bool stream_out) {
    constexpr int NSTG = (NP + 7) / 8, NOUT = TM * 2;
    const int split = (static_cast<int>(blockIdx.x) >> 3) % nsplit;
    const int64_t wave_id = ((static_cast<int64_t>(blockIdx.x) >> 3) / nsplit) * 8 + (blockIdx.x & 7);
    const int64_t nwaves = gridDim.x / nsplit;
    uint16_t* __restrict__ C = C_all + split * (TM * 32);
    const int K = WHOLE ? 16 * NP : K_arg, G = K / 8, pitchB = 2 * K + 8;
    const int AW = WHOLE || Adim_all - split * (TM * 32) >= TM * 32 ? TM * 32 : Adim_all - split * (TM * 32);
    const int UPR = AW / 8, pitchC = 2 * AW + 8;
    extern __shared__ u32x4 smem_u4[];
    // positions of the columns (Eq. (10)'s gather; byte offsets inside a row), then the token rows, later the output rows
    int32_t* sInv = reinterpret_cast<int32_t*>(smem_u4);
    uint8_t* area = reinterpret_cast<uint8_t*>(smem_u4) + (PERM ? NSTG * 512 : 0);
    const int lane = threadIdx.x, l32 = lane & 31, h = lane >> 5;
    // piece lane + 64 it of a tile is piece g of row r; the walk from one `it` to the next adds 64 = dr G + dg
    const int rB = lane / G, gB = lane - rB * G, drB = 64 / G, dgB = 64 - drB * G;
    const int rC = lane / UPR, gC = lane - rC * UPR, drC = 64 / UPR, dgC = 64 - drC * UPR;
    const int64_t ntiles = ceil_div(T, 32);
    int64_t tile = wave_id;
    if (tile >= ntiles) return;
    // (The walks start from copies the optimiser cannot see through: hoisted out of the tile loop, the addresses of all pieces
    // would occupy a few dozen registers for the whole kernel.  Whole pieces need fewer, and have them but in the largest instance.)
    constexpr bool HIDE = !WHOLE || TM * NP >= 40;

    u32x4 v[NP];
    auto load = [&](int64_t tl) {
        const int64_t t0 = tl * 32;
        const int last = static_cast<int>(T - t0 < 32 ? T - t0 : 32) - 1;
        const uint8_t* base = reinterpret_cast<const uint8_t*>(Bsrc + t0 * ldb);
        int r = rB, g = gB;
        if constexpr (HIDE) asm volatile("" : "+v"(r), "+v"(g));       // see above
#pragma unroll
        for (int it = 0; it < NP; ++it) {
            v[it] = *reinterpret_cast<const u32x4*>(base + static_cast<uint32_t>((r < last ? r : last) * (2 * ldb) + 16 * g));
            r += drB; g += dgB;
            if (dgB != 0 && g >= G) { g -= G; r += 1; }
        }
    };
    load(tile);
    u32x4 ra[NSTG][TM][4];
    u32x2 rmeta[NSTG][TM];
    const int rt_last = (Adim_all + 31) / 32 - 1;            // row tiles beyond it re-read it (computed, never stored)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int rt = WHOLE || split * TM + i < rt_last ? split * TM + i : rt_last;
        const uint16_t* pa = A_all + (static_cast<int64_t>(rt) * NSTG * 256 + lane) * 8;
        const uint32_t* pm = Ameta_all + (static_cast<int64_t>(rt) * NSTG * 64 + lane) * 2;
#pragma unroll
        for (int st = 0; st < NSTG; ++st) {
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4)
                ra[st][i][s4] = *reinterpret_cast<const u32x4*>(pa + (st * 4 + s4) * 512);
            rmeta[st][i] = *reinterpret_cast<const u32x2*>(pm + st * 128);
        }
    }
    if constexpr (PERM) {                                    // column c = P[r] goes to position r
        for (int r = lane; r < K; r += 64) sInv[perm[r]] = 2 * r;
    }

    auto put = [&]() {                                       // registers -> LDS rows
        wave_lds_fence();                                    // the previous tile's output rows have been read
        int r = rB, g = gB;
        if constexpr (HIDE) asm volatile("" : "+v"(r), "+v"(g));
#pragma unroll
        for (int it = 0; it < NP; ++it) {
            uint8_t* row = area + (WHOLE || r < 32 ? r : 32) * pitchB;
            if constexpr (PERM) {
                const u32x4 i0 = *reinterpret_cast<const u32x4*>(sInv + 8 * g);
                const u32x4 i1 = *reinterpret_cast<const u32x4*>(sInv + 8 * g + 4);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    *reinterpret_cast<uint16_t*>(row + (e < 4 ? i0[e & 3] : i1[e & 3])) = static_cast<uint16_t>(v[it][e >> 1] >> (16 * (e & 1)));
            } else {
                u32x2* d = reinterpret_cast<u32x2*>(row + 16 * g);
                d[0] = (u32x2){v[it].x, v[it].y};
                d[1] = (u32x2){v[it].z, v[it].w};
            }
            r += drB; g += dgB;
            if (dgB != 0 && g >= G) { g -= G; r += 1; }
        }
        wave_lds_fence();
    };
    // products of the tile in LDS, output rows regrouped through the same area
    auto multiply = [&](int64_t tl, auto last_c) {
        f32x16 acc[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][q] = 0.f;
        const uint8_t* myrow = area + l32 * pitchB + 16 * h;
#pragma unroll
        for (int st = 0; st < NSTG; ++st) {
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                BFragN bf;
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    bf.q[x] = (u32x4){0u, 0u, 0u, 0u};
                    const int g = 16 * st + 8 * x + 2 * s4;  // granules g and g + 1 (one per lane half); the weights beyond K are zero
                    if (g < 2 * NP) {
                        const u32x2* p = reinterpret_cast<const u32x2*>(myrow + 16 * g);
                        const u32x2 lo = p[0], hi = p[1];
                        const bool in = WHOLE || st + 1 < NSTG || g + h < G;
                        bf.q[x] = in ? (u32x4){lo.x, lo.y, hi.x, hi.y} : (u32x4){0u, 0u, 0u, 0u};
                    }
                }
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    AFragN af;
                    af.q = ra[st][i][s4];
                    const int idx = static_cast<int>(s4 < 2 ? rmeta[st][i].x : rmeta[st][i].y);
                    if (s4 & 1)
                        acc[i] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, bf.v, acc[i], idx, 0, 1);
                    else
                        acc[i] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, bf.v, acc[i], idx, 0, 0);
                }
            }
        }
        wave_lds_fence();                                    // all fragment reads precede the overwrite
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const uint32_t xlo = pack_bf16(acc[i][8 * p + 0], acc[i][8 * p + 1]);
                const uint32_t xhi = pack_bf16(acc[i][8 * p + 2], acc[i][8 * p + 3]);
                const uint32_t ylo = pack_bf16(acc[i][8 * p + 4], acc[i][8 * p + 5]);
                const uint32_t yhi = pack_bf16(acc[i][8 * p + 6], acc[i][8 * p + 7]);
                const auto slo = __builtin_amdgcn_permlane32_swap(xlo, ylo, false, false);
                const auto shi = __builtin_amdgcn_permlane32_swap(xhi, yhi, false, false);
                const int a0 = i * 32 + 16 * p + 8 * h;      // first of this lane's 8 weight rows
                if (WHOLE || a0 + 8 <= AW) {
                    u32x2* d = reinterpret_cast<u32x2*>(area + l32 * pitchC + 2 * a0);
                    d[0] = (u32x2){slo[0], shi[0]};
                    d[1] = (u32x2){slo[1], shi[1]};
                }
            }
        wave_lds_fence();
        const int64_t t0 = tl * 32;
        uint8_t* base = reinterpret_cast<uint8_t*>(C + t0 * ldc);
        u32x4 o[NOUT];
        int r = rC, g = gC;
        if constexpr (HIDE) asm volatile("" : "+v"(r), "+v"(g));
#pragma unroll
        for (int it = 0; it < NOUT; ++it) {
            const bool in = WHOLE || r < 32;
            const u32x2* p = reinterpret_cast<const u32x2*>(area + (in ? r : 31) * pitchC + 16 * (in ? g : UPR - 1));
            const u32x2 lo = p[0], hi = p[1];
            o[it] = (u32x4){lo.x, lo.y, hi.x, hi.y};
            r += drC; g += dgC;
            if (dgC != 0 && g >= UPR) { g -= UPR; r += 1; }
        }
        auto emit = [&](bool stream) {
            int re = rC, ge = gC;
            if constexpr (HIDE) asm volatile("" : "+v"(re), "+v"(ge));
#pragma unroll
            for (int it = 0; it < NOUT; ++it) {
                const bool in = WHOLE || re < 32;
                const int rr = in ? re : 31;
                u32x4* dst = reinterpret_cast<u32x4*>(base + static_cast<uint32_t>(rr * (2 * ldc) + 16 * (in ? ge : UPR - 1)));
                if (!decltype(last_c)::value || t0 + rr < T) store16(o[it], dst, stream);
                re += drC; ge += dgC;
                if (dgC != 0 && ge >= UPR) { ge -= UPR; re += 1; }
            }
        };
        if (stream_out) emit(true);
        else emit(false);
    };

    // (a branch around the loads alone would copy their registers where it joins, and wait for them there; the weights are waited
    // for here, vmcnt(0), or every tile would wait for the previous one's stores before it uses them)
    put();
    __builtin_amdgcn_s_waitcnt(0x0F70);
    for (int64_t next = tile + nwaves; next < ntiles; next += nwaves) {
        load(next);                                          // in flight during this tile's arithmetic
        multiply(tile, std::false_type{});
        tile = next;
        put();
    }
    multiply(tile, std::true_type{});
}

// Wavefronts per CU by LDS and registers; the grid is a multiple of the CU count in which every wavefront gets the same number of
// tiles (+-1).  (The occupancy depends on the kernel, the LDS size and the device: remembered per instantiation and device, LDS
// size and answer in one word.)
template <typename Kern>
int narrow_grid(Kern kern, DeviceMemo& memo, int lds, int nsplit, int64_t T, unsigned& grid) {
    const int dev = DeviceMemo::device();
    const uint64_t known = memo.get(dev);
    int wpc = (known >> 32) == static_cast<uint64_t>(lds) ? static_cast<int>(known & 0xFFFFFFFFu) : 0;
    if (wpc < 1) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&wpc, reinterpret_cast<const void*>(kern), 64, static_cast<size_t>(lds)) != hipSuccess || wpc < 1)
            return BIMASK_ERR_HIP;
        memo.set(dev, (static_cast<uint64_t>(lds) << 32) | static_cast<uint32_t>(wpc));
    }
    if (wpc > 16) wpc = 16;
    const int64_t ntiles = ceil_div(T, 32);
    const int64_t slots = 256 * wpc / nsplit;                                   // token tiles in flight on the chip
    const int64_t rounds = ceil_div(ntiles, slots);
    int64_t nwaves = ceil_div(ceil_div(ntiles, rounds), 256) * 256;
    if (nwaves > round_up(ntiles, 8)) nwaves = round_up(ntiles, 8);
    grid = static_cast<unsigned>(nwaves * nsplit);
    return BIMASK_OK;
}

template <int TM, int NSTG>
int run_narrow(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, const void* Bsrc, int64_t ldb,
               const int32_t* perm, int64_t T, void* C, int64_t ldc, hipStream_t s) {
    auto kern = k_gemm_sp24_narrow<TM, NSTG>;
    const int in_bytes = 32 * narrow_pitch(static_cast<int>(K)) + NSTG * 256;   // fragment reads may run past row 31
    const int out_bytes = 32 * narrow_pitch(static_cast<int>(Adim < TM * 32 ? Adim : TM * 32)) + 16;
    const int lds = NSTG * 512 + (((in_bytes > out_bytes ? in_bytes : out_bytes) + 15) & ~15);
    if (lds > 48 * 1024) return BIMASK_ERR_UNSUPPORTED;
    const int nsplit = static_cast<int>(ceil_div(Adim, TM * 32));
    static DeviceMemo memo;
    unsigned grid;
    if (int rc = narrow_grid(kern, memo, lds, nsplit, T, grid)) return rc;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64), static_cast<size_t>(lds), s, static_cast<const uint16_t*>(A), meta,
                       static_cast<int>(Adim), static_cast<int>(K), static_cast<const uint16_t*>(Bsrc),
                       static_cast<int>(ldb), perm, T, static_cast<uint16_t*>(C), static_cast<int>(ldc), nsplit,
                       streams_out(C, Adim, ldc, nsplit == 1));
    return check_launch();
}

template <int TM, int NP, bool PERM, bool WHOLE>
int run_narrow_rows(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, const void* Bsrc, int64_t ldb, const int32_t* perm,
                    int64_t T, void* C, int64_t ldc, hipStream_t s) {
    auto kern = k_gemm_sp24_narrow_rows<TM, NP, PERM, WHOLE>;
    const int k = static_cast<int>(K), a = static_cast<int>(Adim < TM * 32 ? Adim : TM * 32);
    const int in_bytes = (WHOLE ? 32 : 33) * (2 * k + 8) + 256, out_bytes = 32 * (2 * a + 8);      // fragment reads may run past row 31
    const int lds = (PERM ? (NP + 7) / 8 * 512 : 0) + (((in_bytes > out_bytes ? in_bytes : out_bytes) + 15) & ~15);
    const int nsplit = static_cast<int>(ceil_div(Adim, TM * 32));
    static DeviceMemo memo;
    unsigned grid;
    if (int rc = narrow_grid(kern, memo, lds, nsplit, T, grid)) return rc;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64), static_cast<size_t>(lds), s, static_cast<const uint16_t*>(A), meta,
                       static_cast<int>(Adim), k, static_cast<const uint16_t*>(Bsrc), static_cast<int>(ldb), perm, T,
                       static_cast<uint16_t*>(C), static_cast<int>(ldc), nsplit, streams_out(C, Adim, ldc, nsplit == 1));
    return check_launch();
}

}  // namespace

// Whole pieces and whole row tiles (us, column tiles -> here: 256 -> 32 columns at 5212 tokens 4.1 -> 3.7, at 122211 17.7 -> 15.8; 256
// -> 64 at 20709 6.3 -> 5.4, at 200704 32.8 -> 28.8, from 96 tiles on: at 1509 3.7 / 3.8; ragged, 256 -> 56 at 20000 5.8 / 6.6).
// A second stage that is nearly all padding, one row tile and many tokens, where column tiles of 64 tokens are many short rounds
// (144 -> 32 at 246298 29.7 -> 24.0, 136 -> 16 at 333432 36.6 -> 26.7, 160 -> 32 at 164190 21.2 -> 19.4; at 53342, 160 -> 8, 9.0 / 8.2
// in cache and 9.4 / 9.5 from memory, 192 -> 32 at 197689 24.1 / 24.9).
bool gemm_sp24_narrow_streams(int64_t Adim, int64_t K, int64_t T) {
    if (K == 256) return Adim == 32 || (Adim == 64 && T >= 3072);
    return K > 128 && K <= 160 && Adim <= 32 && T >= 49152;
}

// Returns BIMASK_ERR_UNSUPPORTED when the shape, the alignment or the leading dimensions are
// outside what this kernel handles (the caller then takes the workgroup-tiled kernels).
int launch_gemm_sp24_narrow(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, const void* Bsrc,
                            int64_t ldb, const int32_t* perm, int64_t T, void* C, int64_t ldc, hipStream_t s) {
    if (T < 1 || K < 4 || Adim < 4 || K % 4 != 0 || Adim % 4 != 0) return BIMASK_ERR_UNSUPPORTED;
    if (!aligned16(A) || !aligned16(meta) || !aligned16(Bsrc) || !aligned16(C)) return BIMASK_ERR_UNSUPPORTED;
    if (ldb >= (1 << 20) || ldc >= (1 << 20)) return BIMASK_ERR_UNSUPPORTED;    // 32-bit offsets inside a tile
    if (K % 8 != 0 ? (ldb != K || perm) : ldb % 8 != 0) return BIMASK_ERR_UNSUPPORTED;
    if (Adim % 8 != 0 ? ldc != Adim : ldc % 8 != 0) return BIMASK_ERR_UNSUPPORTED;
    const int nstg = static_cast<int>(ceil_div(K, 128)), tm = static_cast<int>(ceil_div(Adim, 32));
    // six row tiles and more go to two wavefronts, which both read the token rows: not with dX on top of dY
    if (perm && tm > 5 && !disjoint(Bsrc, T, ldb, K, C, ldc, Adim, 2)) return BIMASK_ERR_UNSUPPORTED;
// WHOLE where the pieces fill an instance (K = 16 NP) and the weight rows its row tiles: every walk over pieces has constant steps
    // (K = 64 and 128 on 32 .. 256 columns, us, ragged form -> whole: 96 <- 128 at 7003 tokens 3.95 -> 3.0, 128 -> 32 with the gather at
    // 121643 9.03 -> 7.4, 160 <- 64 at 31836 5.63 -> 4.8, from 0.70 of the ragged time at 4000 tokens to 0.97 at 400000).
#define BIMASK_ROWS_FORM(TM_, NP_, P_, PERM_)                                                                         \
    return K == 16 * NP_ && Adim % (32 * TM_) == 0 ? run_narrow_rows<TM_, NP_, P_, true>(A, meta, Adim, K, Bsrc, ldb, PERM_, T, C, ldc, s)  \
                                                   : run_narrow_rows<TM_, NP_, P_, false>(A, meta, Adim, K, Bsrc, ldb, PERM_, T, C, ldc, s);
#define BIMASK_ROWS(TM_, NP_) { if (perm) BIMASK_ROWS_FORM(TM_, NP_, true, perm) BIMASK_ROWS_FORM(TM_, NP_, false, nullptr) }
#define BIMASK_ROWS_PLAIN(TM_, NP_) return run_narrow_rows<TM_, NP_, false, false>(A, meta, Adim, K, Bsrc, ldb, nullptr, T, C, ldc, s);
    if (K % 8 == 0 && Adim % 8 == 0) {
        if (nstg == 1) {
#define BIMASK_ROWS_TILES(NP_)                                                                                        \
            switch (tm) {                                                                                             \
                case 1: BIMASK_ROWS(1, NP_)                                                                           \
                case 2: BIMASK_ROWS(2, NP_)                                                                           \
                case 3: case 6: BIMASK_ROWS(3, NP_)          /* six to eight row tiles: two wavefronts per token tile */ \
                case 4: case 7: case 8: BIMASK_ROWS(4, NP_)                                                           \
                case 5: BIMASK_ROWS(5, NP_)                                                                           \
                default: break;                                                                                       \
            }
            if (K <= 64) BIMASK_ROWS_TILES(4) else BIMASK_ROWS_TILES(8)
#undef BIMASK_ROWS_TILES
        } else if (perm) {                                   // longer contractions with the gather: column tiles, but for these
            if (!gemm_sp24_narrow_streams(Adim, K, T)) return BIMASK_ERR_UNSUPPORTED;
            if (K < 256) return run_narrow<1, 2>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, s);
            if (tm == 1) return run_narrow_rows<1, 16, true, true>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, s);
            return run_narrow_rows<2, 16, true, true>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, s);
        } else if (tm <= 2 || (tm <= 4 && nstg == 2 && T >= (K < 256 || Adim == 128 ? 16384 : 98304))) {
            // Longer contractions: at most 64 weight rows, all their fragments in registers.  Up to 128 rows on two wavefronts per token
            // tile gain with two stages and many tokens: below 256 terms against the resident kernel (224 -> 88 columns at 30096
            // tokens 10.1 -> 7.6 us), at 256 against the streaming one, with whole row tiles (256 -> 128 at 18762 5.3 -> 4.9, at 73446
            // 12.6 -> 9.9, at 180062 25.0 -> 22.8) sooner than with ragged ones (256 -> 104 at 44161 7.5 / 10.0, at 106868 17.5 / 17.5).
            switch (nstg) {
                case 2: if (tm == 1) BIMASK_ROWS_FORM(1, 16, false, nullptr) else BIMASK_ROWS_FORM(2, 16, false, nullptr)
                case 3: if (tm == 1) BIMASK_ROWS_PLAIN(1, 24) else BIMASK_ROWS_PLAIN(2, 24)
                case 4: if (tm == 1) BIMASK_ROWS_PLAIN(1, 32) else BIMASK_ROWS_PLAIN(2, 32)
                default: break;
            }
        }
        return BIMASK_ERR_UNSUPPORTED;
    }
#undef BIMASK_ROWS_PLAIN
#undef BIMASK_ROWS
#undef BIMASK_ROWS_FORM
#define BIMASK_NARROW(TM_, NSTG_) return run_narrow<TM_, NSTG_>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, s);
    if (nstg == 1) {
        switch (tm) {
            case 1: BIMASK_NARROW(1, 1)
            case 2: BIMASK_NARROW(2, 1)
            case 3: BIMASK_NARROW(3, 1)
            case 4: BIMASK_NARROW(4, 1)
            case 5: BIMASK_NARROW(5, 1)
            default: break;
        }
        // up to 256 weight rows: two wavefronts per token tile, each with half of the rows (the
        // token rows are short, so fetching them twice from L2 is cheap next to the output)
        if (Adim % 8 == 0) {
            if (tm == 6) BIMASK_NARROW(3, 1)
            if (tm == 7 || tm == 8) BIMASK_NARROW(4, 1)
        }
    } else if (tm <= 2) {
        // longer contractions: at most 64 weight rows, all their fragments in registers.  (Splitting
        // more rows over sibling wavefronts does not pay here: every sibling re-reads the long rows.)
        switch (nstg) {
            case 2: if (tm == 1) BIMASK_NARROW(1, 2) else BIMASK_NARROW(2, 2)
            case 3: if (tm == 1) BIMASK_NARROW(1, 3) else BIMASK_NARROW(2, 3)
            case 4: if (tm == 1) BIMASK_NARROW(1, 4) else BIMASK_NARROW(2, 4)
            default: break;
        }
    }
#undef BIMASK_NARROW
    return BIMASK_ERR_UNSUPPORTED;
}

}  // namespace bimask
