// N:M-sparse bf16 GEMM for wide outputs and contractions up to 512 terms (arXiv 2302.06058, Eq. (3) and Eq. (10)):
//     C[t][a] = sum_k Bsrc[t][perm[k]] * A[a][k]
//
// A workgroup loads its token tile once (64 or 128 whole rows, granules XOR-swizzled as in the streaming kernel; Eq. (10)'s gather
// is a 2-byte scatter on the way in) and its eight wavefronts then work on their own: each takes pairs of weight-row tiles (64
// rows) in turn against ALL tokens of the tile, weights from L2 into registers that are re-loaded as soon as they are used, and
// writes its 64 columns through an LDS strip of its own as whole 128-byte lines.  No barrier after the fill, so one wavefront's
// output overlaps another's products (not its own: its next tile waits for weights requested before its stores).  The weight-row-tile loop of the resident kernel (32 rows per wavefront, a barrier per
// 256) reads every token fragment from LDS for one matrix instruction; here it serves two, and with 128 tokens a weight fragment
// serves four: half the LDS reads and half the weight bytes through the CU.
// Measured, us (resident or streaming -> here; means over four cards, buffers in turn): 384 -> 1536 columns with the gather at 25216
// tokens 45.2 -> 33.1, without 38.4 -> 30.0, 4:8 47.4 -> 37.5; 384 -> 1152 29.3 -> 21.7.  What bounds it (timestamps, 384 -> 1536): 8 us
// until the rows are in LDS, then 5.7 per 64 x 100 tile of a wavefront, half of it its output (4 TB/s over the chip).
#include "common.hpp"

namespace bimask {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(__bf16)))) __bf16 bf16x16;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

union BFragV { bf16x16 v; bf16x8 half[2]; u32x4 q[2]; };
union AFragV { bf16x8 v; u32x4 q; };

constexpr int kWideLds = 160 * 1024;
constexpr int kWideWaves = 8;
constexpr int kWideStage = 32 * 136;                     // output staging of a wavefront: 32 tokens x 64 weight rows

// TN: token sub-tiles of 32 in a tile.  DENSE: the dense masked operand of a ratio with N > 2, two 32x32x16 instructions per sparse
// 32x32x32 and weight steps of 64 contraction indices.  blockIdx.y: pieces of `wpp` wavefront tiles (64 weight rows each).
template <int TN, bool DENSE>
__global__ void __launch_bounds__(64 * kWideWaves, 2)
k_gemm_sp24_wide(const uint16_t* __restrict__ A, const uint32_t* __restrict__ Ameta, int Adim, int K,
                 const uint16_t* __restrict__ Bsrc, int64_t ldb, const int32_t* __restrict__ perm, int64_t T,
                 uint16_t* __restrict__ C, int64_t ldc, int rpt, int wpp, bool stream_out) {
    constexpr int NWV = kWideWaves, NT = 64 * NWV, TM = 2, ROWS = 32 * TN;
    constexpr int SUB = DENSE ? 2 : 4, NX = 4 / SUB;     // sub-steps of a weight step; fragments per row tile and sub-step
    extern __shared__ u32x4 smem_u4[];
    uint8_t* smem = reinterpret_cast<uint8_t*>(smem_u4);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int nks = (K + 127) >> 7, nst = DENSE ? 2 * nks : nks;
    const int ntr = (Adim + 31) >> 5, nwt = (ntr + 1) >> 1;              // row tiles, wavefront tiles of two
    uint8_t* sOut = smem + nks * (ROWS * 256) + wave * kWideStage;
    uint16_t* sInv = reinterpret_cast<uint16_t*>(smem + nks * (ROWS * 256) + NWV * kWideStage);
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * rpt;
    const int rows = static_cast<int>(T - t0 < rpt ? T - t0 : rpt);
    int wt = static_cast<int>(blockIdx.y) * wpp + wave;                                    // this wavefront's tiles: wt, wt + NWV, ...
    const int wt_all = (static_cast<int>(blockIdx.y) + 1) * wpp, wt_end = wt_all < nwt ? wt_all : nwt;

    // ---- weights: step `ws` of tile `ww` is the next to request
    const uint32_t lane16 = lane * 16, lane8 = lane * 8;
    u32x4 ra[TM][4];
    u32x2 rmn[DENSE ? 1 : TM];
    int ww = wt < wt_end ? wt : wt_end - 1, ws = 0;
    auto row_tile = [&](int i) { const int rt = 2 * ww + i; return rt < ntr ? rt : ntr - 1; };       // clamped: computed, never stored
    auto weights = [&](int i) { return reinterpret_cast<const uint8_t*>(A) + (static_cast<int64_t>(row_tile(i)) * nst + ws) * 4096; };
    auto index = [&](int i) { return reinterpret_cast<const uint8_t*>(Ameta) + (static_cast<int64_t>(row_tile(i)) * nks + ws) * 512; };
    auto advance = [&]() {
        const bool wrap = ws + 1 == nst;
        ws = wrap ? 0 : ws + 1;
        ww = wrap && ww + NWV < wt_end ? ww + NWV : ww;
    };
    if constexpr (!DENSE)
#pragma unroll
        for (int i = 0; i < TM; ++i) rmn[i] = *reinterpret_cast<const u32x2*>(index(i) + lane8);
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int i = 0; i < TM; ++i) ra[i][g] = *reinterpret_cast<const u32x4*>(weights(i) + g * 1024 + lane16);
    advance();

    // ---- token rows: 16-byte pieces into granules (8 columns) that are XOR-swizzled by the row.  Unconditional (pieces beyond the
    // tile repeat its last row), in groups of four: all in flight at once, where a wait per conditional load would line them up.
    {
        const int G = K >> 3, total = rows * G;
        constexpr int U = 16;                                            // pieces of a thread, at most
        const int dt = NT / G, dg = NT - dt * G;
        int t = tid / G, g = tid - t * G;
        u32x4 v[U];
        int tt[U], gg[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            tt[u] = t < rows ? t : rows - 1; gg[u] = g;
            t += dt; g += dg;
            if (g >= G) { g -= G; t += 1; }
        }
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += 4)
            if (NT * u0 < total) {
#pragma unroll
                for (int u = u0; u < u0 + 4; ++u) v[u] = *reinterpret_cast<const u32x4*>(Bsrc + (t0 + tt[u]) * ldb + 8 * gg[u]);
            }
        if (perm) {                                                      // uniform
            for (int r = tid; r < K; r += NT) sInv[perm[r]] = static_cast<uint16_t>(r);
            __syncthreads();
        }
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += 4)
            if (NT * u0 < total) {
#pragma unroll
                for (int u = u0; u < u0 + 4; ++u) {
                    uint8_t* row = smem + tt[u] * 256;
                    const int sw = tt[u] & 15;
                    if (perm) {                                          // Eq. (10)'s column gather: column c = P[r] goes to position r
                        const u32x4 iv = *reinterpret_cast<const u32x4*>(sInv + 8 * gg[u]);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int pos = (iv[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
                            *reinterpret_cast<uint16_t*>(row + (pos >> 7) * (ROWS * 256) + ((((pos & 127) >> 3) ^ sw) << 4) + 2 * (pos & 7)) =
                                static_cast<uint16_t>(v[u][e >> 1] >> (16 * (e & 1)));
                        }
                    } else {
                        *reinterpret_cast<u32x4*>(row + (gg[u] >> 4) * (ROWS * 256) + (((gg[u] & 15) ^ sw) << 4)) = v[u];
                    }
                }
            }
        if (K & 127) {                                                   // granules that only the padding of the weights has
            const int gl = (K & 127) >> 3, n = 16 - gl;
            for (int c = tid; c < ROWS * n; c += NT) {
                const int tr = c / n, gp = gl + c - tr * n;
                *reinterpret_cast<u32x4*>(smem + (nks - 1) * (ROWS * 256) + tr * 256 + ((gp ^ (tr & 15)) << 4)) = (u32x4){0u, 0u, 0u, 0u};
            }
        }
    }
    __syncthreads();
    if (wt >= wt_end) return;

    f32x16 acc[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
    };
    clear();
    int fo[4][2];                                                        // granule of k = 32 s4 + 8 h + 64 x in the row of token l32
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
        for (int x = 0; x < 2; ++x) fo[s4][x] = l32 * 256 + (((8 * x + 2 * s4 + h) ^ (l32 & 15)) << 4);
    constexpr int kDepth = 3, NQ = 4 * TN;                               // fragments read ahead; fragments of a stage
    BFragV f[kDepth + 1];
    auto read = [&](int stage, int q) {                                  // fragment q of a stage: sub-step q / TN, tokens 32 (q % TN) ..
        const uint8_t* p = smem + stage * (ROWS * 256) + (q % TN) * 8192;
        f[q % (kDepth + 1)].q[0] = *reinterpret_cast<const u32x4*>(p + fo[q / TN][0]);
        f[q % (kDepth + 1)].q[1] = *reinterpret_cast<const u32x4*>(p + fo[q / TN][1]);
    };
    static_assert(NQ % (kDepth + 1) == 0, "the fragment ring runs over stages");
#pragma unroll
    for (int q = 0; q < kDepth; ++q) read(0, q);
    int st = 0;
#pragma unroll 1
    for (;;) {
        u32x2 m[DENSE ? 1 : TM];
        uint32_t l16 = lane16, l8 = lane8;
        asm volatile("" : "+v"(l16), "+v"(l8));
        if constexpr (!DENSE) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                m[i] = rmn[i];
                rmn[i] = *reinterpret_cast<const u32x2*>(index(i) + l8);
            }
        }
        const int st_next = st + 1 < nks ? st + 1 : 0;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const uint8_t* wb[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) wb[i] = weights(i);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int q = s4 * TN + j;
                read(q + kDepth < NQ ? st : st_next, (q + kDepth) % NQ);
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const BFragV& b = f[q % (kDepth + 1)];
                    AFragV af;
                    if constexpr (DENSE) {
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            af.q = ra[i][2 * (s4 & 1) + x];
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af.v, b.half[x], acc[i][j], 0, 0, 0);
                        }
                    } else {
                        af.q = ra[i][s4];
                        const int idx = static_cast<int>(s4 < 2 ? m[i].x : m[i].y);
                        if (s4 & 1) acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, b.v, acc[i][j], idx, 0, 1);
                        else acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, b.v, acc[i][j], idx, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // the registers just used take the same place of the next step
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int x = 0; x < NX; ++x) {
                    const int g = (s4 % SUB) * NX + x;
                    ra[i][g] = *reinterpret_cast<const u32x4*>(wb[i] + g * 1024 + l16);
                }
            if (s4 % SUB == SUB - 1) advance();
            __builtin_amdgcn_sched_barrier(0);
        }
        st = st_next;
        if (st == 0) {
            // a tile is done: 32 tokens x 64 weight rows at a time through the wavefront's own staging rows
            const int a0 = wt * 64;
            // (Uniform row addresses and one 32-bit offset per lane: with a 64-bit address per store and lane the 128-token tile of
            // 2-of-4 weights spilled two registers, and their reload waited for every load and store in flight.  384 -> 1152 columns
            // at 25216 tokens 21.7 -> 21.2 us, 52 shapes of this instance 1.4 % faster in the mean, the others 0.4 to 0.9 %.)
            const uint32_t out_ofs = static_cast<uint32_t>(lane >> 3) * (2 * static_cast<uint32_t>(ldc)) + 16 * (lane & 7);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (32 * j < rows) {                                     // uniform
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            const uint32_t xlo = pack_bf16(acc[i][j][8 * p + 0], acc[i][j][8 * p + 1]);
                            const uint32_t xhi = pack_bf16(acc[i][j][8 * p + 2], acc[i][j][8 * p + 3]);
                            const uint32_t ylo = pack_bf16(acc[i][j][8 * p + 4], acc[i][j][8 * p + 5]);
                            const uint32_t yhi = pack_bf16(acc[i][j][8 * p + 6], acc[i][j][8 * p + 7]);
                            const auto slo = __builtin_amdgcn_permlane32_swap(xlo, ylo, false, false);
                            const auto shi = __builtin_amdgcn_permlane32_swap(xhi, yhi, false, false);
                            u32x2* d = reinterpret_cast<u32x2*>(sOut + l32 * 136 + 2 * (32 * i + 16 * p + 8 * h));
                            d[0] = (u32x2){slo[0], shi[0]};
                            d[1] = (u32x2){slo[1], shi[1]};
                        }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    u32x4 o[4];
#pragma unroll
                    for (int it = 0; it < 4; ++it) {
                        const u32x2* p = reinterpret_cast<const u32x2*>(sOut + ((lane >> 3) + 8 * it) * 136 + 16 * (lane & 7));
                        const u32x2 lo = p[0], hi = p[1];
                        o[it] = (u32x4){lo.x, lo.y, hi.x, hi.y};
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
                    for (int it = 0; it < 4; ++it) {
                        const int t = 32 * j + 8 * it;
                        uint8_t* row = reinterpret_cast<uint8_t*>(C + (t0 + t) * ldc + a0);
                        if ((lane >> 3) < rows - t && 8 * (lane & 7) < Adim - a0)        // Adim is a multiple of 8
                            store16(o[it], reinterpret_cast<u32x4*>(row + out_ofs), stream_out);
                    }
                }
            }
            wt += NWV;
            if (wt >= wt_end) break;
            clear();
        }
    }
}

struct WidePlan { int tn, rpt, wpp; unsigned grid, pieces; size_t lds; };

// Tokens per workgroup and pieces of weight rows for tiles of 32 tn tokens: as many pieces as still fit one round of 256 workgroups,
// then the lowest tile that needs no more rounds.  Returns the estimated time (us; fitted within 25 % to 320 timed launches, over
// which the choice between 64 and 128 tokens costs 1-2 % against the better one), 0 where the tile does not fit.
double wide_plan(int tn, int64_t Adim, int64_t K, int64_t T, bool perm, bool dense, WidePlan& p) {
    const int64_t nks = ceil_div(K, 128), nwt = ceil_div(Adim, 64);
    p.lds = static_cast<size_t>(nks * (32 * tn * 256) + kWideWaves * kWideStage + (perm ? round_up(2 * K, 16) : 0));
    if (p.lds > kWideLds || 4 * tn * K > 16 * 64 * kWideWaves) return 0;           // LDS; pieces of a fetching thread
    int64_t pieces = 256 / ceil_div(T, 32 * tn);
    pieces = pieces < 1 ? 1 : pieces > nwt ? nwt : pieces;
    const int64_t slots = 256 / pieces, rounds = ceil_div(ceil_div(T, 32 * tn), slots);
    const int64_t low = ceil_div(T, slots * rounds);
    p.tn = tn;
    p.rpt = static_cast<int>(low < 32 * tn ? low : 32 * tn);
    p.wpp = static_cast<int>(ceil_div(nwt, pieces));
    p.grid = static_cast<unsigned>(ceil_div(T, p.rpt));
    p.pieces = static_cast<unsigned>(ceil_div(nwt, p.wpp));
    const double scatter = perm ? p.rpt * K / 1e4 : 0, steps = static_cast<double>(ceil_div(p.wpp, kWideWaves) * nks);
    const double out = static_cast<double>(ceil_div(p.wpp, kWideWaves)) * p.rpt / 100;
    if (tn == 4) return dense ? rounds * (0.19 + 1.14 * scatter + 2.19 * steps + 4.14 * out) : rounds * (2.21 + 0.74 * scatter + 1.68 * steps + 3.10 * out);
    return dense ? rounds * (1.71 + 1.40 * scatter + 1.18 * steps + 4.45 * out) : 0.53 + rounds * (2.07 + 0.91 * scatter + 0.84 * steps + 3.73 * out);
}

template <int TN, bool DENSE>
int run_wide(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, const void* Bsrc, int64_t ldb, const int32_t* perm,
             int64_t T, void* C, int64_t ldc, const WidePlan& p, hipStream_t s) {
    auto kern = k_gemm_sp24_wide<TN, DENSE>;
    static DeviceMemo attr_set;
    const int dev = DeviceMemo::device();
    if (!attr_set.get(dev)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kWideLds) != hipSuccess)
            return BIMASK_ERR_HIP;
        attr_set.set(dev, 1);
    }
    const bool stream_out = streams_out(C, Adim, ldc, false);
    hipLaunchKernelGGL(kern, dim3(p.grid, p.pieces), dim3(64 * kWideWaves), p.lds, s, static_cast<const uint16_t*>(A), meta,
                       static_cast<int>(Adim), static_cast<int>(K), static_cast<const uint16_t*>(Bsrc), ldb, perm, T,
                       static_cast<uint16_t*>(C), ldc, p.rpt, p.wpp, stream_out);
    return check_launch();
}

}  // namespace

// Returns BIMASK_ERR_UNSUPPORTED where shape or alignment are outside this kernel, or another one is the faster.
int launch_gemm_sp24_wide(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, const void* Bsrc, int64_t ldb,
                          const int32_t* perm, int64_t T, void* C, int64_t ldc, hipStream_t s, bool dense) {
    if (K > 512 || K % 8 != 0 || Adim % 8 != 0 || T > 0x7FFFFFFF) return BIMASK_ERR_UNSUPPORTED;
    if (ldc >= (1 << 28)) return BIMASK_ERR_UNSUPPORTED;                // 32-bit offsets over 8 output rows
    if (!aligned16(A) || !aligned16(meta) || !aligned16(Bsrc) || !aligned16(C) || ldb % 8 != 0 || ldc % 8 != 0)
        return BIMASK_ERR_UNSUPPORTED;
    if (!disjoint(Bsrc, T, ldb, K, C, ldc, Adim, 2)) return BIMASK_ERR_UNSUPPORTED;     // pieces of weight rows read the same tokens
    // Where it gains (700 random shapes, us, old -> here).  2-of-4, above one stage of 128 terms and 256 columns: 160 -> 512 at 20591
    // tokens 12.6 -> 9.6, 384 -> 3008 with the gather at 20856 77.6 -> 50.6, 352 -> 1256 at 3617 9.9 -> 8.1; not 128 -> 2944 at 13325
    // 18.5 / 20.9, 480 -> 320 at 34188 21.4 / 23.1 apart, few tokens (184 -> 3936 at 3185 11.1 / 12.1) where the weight stream counts, and
    // many tokens whose columns cannot stream out (192 -> 2320 at 34405 63.0 / 66.6; 4:8 328 -> 728 at 80233 78.7 / 89.4).  Dense,
    // which has no resident kernel: from 256 columns (160 -> 1360 at 12712 23.1 -> 17.7, with the gather 128 -> 800 at 8244 12.9 ->
    // 10.7; not 192 -> 384 with it at 77300 34.7 / 38.3, which un-permutes the weights instead, 464 -> 1480 at 8649 26.6 / 27.7).
    const bool sectors = Adim % 32 == 0 || (T < 16384 && K > (dense ? 160 : 256));
    const bool gains = dense
        ? K >= 64 && K <= 416 && sectors &&
          ((Adim > 512 && T >= 4096) || (Adim > 256 && T >= 5000 && (!perm || K <= 160)) || (Adim > 1024 && T >= 2048))
        : K > 128 && sectors &&
          ((Adim > 512 && T >= 5000) || (Adim > 256 && T >= 16384) || (Adim > 1024 && K > 256 && T >= 3072));
    if (!gains) return BIMASK_ERR_UNSUPPORTED;
    // Two stages, against the resident kernel where that fills one or two rounds of workgroups: it writes rows in pieces of 256
    // columns, this one in pieces of 64, both ends of which lie inside a 128-byte line where the columns are an odd multiple of 32.
    // 1504 shapes and 191 more; resident -> here with the resident kernel's slots more than 70 % (one round) or 80 % full: 8 % slower in
    // the mean (192 -> 3040 with the gather at 32475 tokens 49.8 / 60.4, 160 -> 3232 at 6665 15.3 / 18.6, 224 -> 3680 without at 16316
    // 31.4 / 37.0); with 43 to 62 % 14 % faster, from 33000 tokens 3 %, at 5000 10 %, columns that are multiples of 64 12 %.
    if (!dense && K <= 256 && Adim % 64 != 0 && Adim > (perm ? 768 : 1024) && T > 5400 && T <= 32768 &&
        gemm_sp24_resident_fill(Adim, T) > (T <= 16384 ? 0.7 : 0.8))
        return BIMASK_ERR_UNSUPPORTED;
    // Four stages, where only tiles of 64 tokens fit: not with a second round just begun (448 -> 384 at 16681 tokens 11.7 / 12.9, 480 -> 640
    // at 18165 18.1 / 19.5, 512 -> 576 at 20953 17.6 / 19.2, but 416 -> 544 at 21834 24.0 -> 19.2; 448 -> 480 at 16421, where the streaming
    // kernel's 256-row tiles are not full, 16.9 -> 14.2; 416 -> 1056 at 19755 32.0 -> 25.7; with the gather always).
    if (!dense && !perm && K > 384 && Adim <= 768 && (Adim <= 384 || Adim > 512) && T > 16384 && T < 21760) return BIMASK_ERR_UNSUPPORTED;
    WidePlan p2, p4;
    const double us2 = wide_plan(2, Adim, K, T, perm != nullptr, dense, p2), us4 = wide_plan(4, Adim, K, T, perm != nullptr, dense, p4);
    if (us2 == 0) return BIMASK_ERR_UNSUPPORTED;
    if (us4 != 0 && us4 < us2)
        return dense ? run_wide<4, true>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p4, s)
                     : run_wide<4, false>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p4, s);
    return dense ? run_wide<2, true>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p2, s)
                 : run_wide<2, false>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p2, s);
}

}  // namespace bimask
