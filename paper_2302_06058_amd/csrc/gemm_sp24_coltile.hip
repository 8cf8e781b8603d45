// N:M-sparse bf16 backward GEMM with the column gather of Eq. (10) fused (arXiv 2302.06058):
//     dX[t][j] = sum_r dY[t][P[r]] * Wb[j][r],   128 < I <= 2048 terms
// on a token tile that lies in LDS COLUMN by column (all its tokens of one out-feature side by side).
//
// Eq. (10) permutes the columns of g(Y).  In a column-major tile that is a permutation of LDS rows: four lanes' worth of a
// token row, transposed in registers (4 tokens x 8 columns, 16 byte-permutes), leaves as eight 8-byte stores whose addresses
// come from the inverse permutation -- where row-major tiles take one 2-byte store per element.  The matrix instructions want
// 8 consecutive contraction indices of one token per lane: the transposing LDS read (ds_read_b64_tr_b16) turns the tile back.
//
// What bounds it is the CU's vector-memory path, through which every token tile pulls the whole weight operand (about 80
// bytes/ns; loads return in order, so rows of g(Y) still on their way from memory hold up the weights behind them).  So the
// tile is as tall as LDS takes (64 tokens up to 1150 columns, 52 of 1536, 36 of 2048) and ONE workgroup owns the CU: wavefronts
// 0-3 multiply, each TM row tiles (32 rows) against all tokens, weights straight from L2 into registers that are re-loaded as
// soon as they are used; wavefronts 4-7 hold the next tile's rows in registers meanwhile.  With 32-row tiles, two workgroups
// per CU and 2-byte stores (before -> now, backward, us; means over four cards, buffers in turn): 1152 x 384 at 25216 tokens 45.6 ->
// 31.2, 4:8 1536 x 384 69.3 -> 48.4, 1024 x 256 at 12544 17.7 -> 14.0, 2048 x 512 at 3136 19.4 -> 12.6; 1504 x 192 at 1100 15.7 -> 7.5;
// where dY was gathered by a pass of its own: 768 x 768 at 8192 23.7 -> 12.8, 2048 x 768 at 3000 30.4 -> 19.2.
// 1152 x 384 took 33 us with plain stores of its output, of which (timestamps inside the kernel): rows of the first tile 7.5, written 1.5, products while the second tile's rows
// arrive 10.5 (6.2 without), output and writing 3, products 6.2, output 1.  Tried without gain: a shorter first tile (33.7),
// the stages in another order per workgroup, the rows pulled into L2 by scalar loads first (46-58).
#include "common.hpp"
#include <type_traits>

namespace bimask {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(__bf16)))) __bf16 bf16x16;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

union BFragT { bf16x16 v; bf16x8 half[2]; u32x2 d[4]; };
union AFragT { bf16x8 v; u32x4 q; };

constexpr int kColThreads = 512;                         // 4 wavefronts multiply, 4 fetch
constexpr int kColUnits = 10;                            // 4-row x 8-column pieces a fetching thread holds, at most
constexpr int kColLds = 160 * 1024;

// 4 consecutive contraction indices of one token per lane out of a column-major tile (16 lanes: 4 columns x 16 tokens)
__device__ __forceinline__ u32x2 read_turned(const uint8_t* p) {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p)));
}

// TM: row tiles per multiplying wavefront; TN: token sub-tiles of 32; NU: pieces of 4 rows x 8 columns per fetching thread.
// DENSE: the weight operand is the dense masked matrix of a ratio with N > 2 (fragment-major): two 16-byte fragments per
// sub-step and two dense 32x32x16 instructions instead of one sparse 32x32x32, steps of 64 contraction indices.
// blockIdx.y: pieces of 128 TM weight rows, where there are fewer token tiles than CUs or more than 384 rows.
template <int TM, int TN, bool DENSE, int NU>
__global__ void __launch_bounds__(kColThreads, 2)
k_gemm_sp24_coltile(const uint16_t* __restrict__ A, const uint32_t* __restrict__ Ameta, int Adim, int K,
                    const uint16_t* __restrict__ Bsrc, int64_t ldb, const int32_t* __restrict__ perm, int64_t T,
                    uint16_t* __restrict__ C, int64_t ldc, int chunk, int rpt, int pitch, bool stream_out) {
    extern __shared__ u32x4 smem_u4[];
    uint8_t* smem = reinterpret_cast<uint8_t*>(smem_u4);
    uint16_t* sInv = reinterpret_cast<uint16_t*>(smem);                  // position of column c in a permuted row
    uint8_t* area = smem + ((2 * K + 15) & ~15);                         // the token tile, later its output rows
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this workgroup's tokens, in tiles of rpt
    const int64_t tok0 = static_cast<int64_t>(blockIdx.x) * chunk;
    const int ntok = static_cast<int>(T - tok0 < chunk ? T - tok0 : chunk);
    Bsrc += tok0 * ldb;
    C += tok0 * ldc;
    const int nks = (K + 127) >> 7;                                      // 128-deep stages of the padded weight operand
    const int ntr = (Adim + 31) >> 5;                                    // 32-row tiles of the weight operand
    const int rtb = blockIdx.y * (4 * TM);                               // first row tile of this workgroup
    const int a_base = rtb * 32;
    const int width = Adim - a_base < 4 * TM * 32 ? Adim - a_base : 4 * TM * 32;
    const int pitchC = 2 * width + 8;

    for (int r = tid; r < K; r += kColThreads) sInv[perm[r]] = static_cast<uint16_t>(r);
    auto clear_tail = [&](int id, int n) {                               // columns that only the padding of the weights has
        for (int b = K * pitch + 8 * id; b < nks * 128 * pitch; b += 8 * n) *reinterpret_cast<u32x2*>(area + b) = (u32x2){0u, 0u};
    };
    auto copy_out = [&](int t0, int end) {
        const int rows = (end < ntok ? end : ntok) - t0;
        const int UPR = width >> 3, total = rows * UPR;
        for (int c = tid; c < total; c += kColThreads) {
            const int t = c / UPR, u = c - t * UPR;
            const u32x2* p = reinterpret_cast<const u32x2*>(area + t * pitchC + 16 * u);
            const u32x2 lo = p[0], hi = p[1];
            const u32x4 o = {lo.x, lo.y, hi.x, hi.y};
            u32x4* dst = reinterpret_cast<u32x4*>(C + (t0 + t) * ldc + a_base + 8 * u);
            store16(o, dst, stream_out);
        }
    };

    if (wave >= 4) {
        // ---- wavefronts 4-7: rows of g(Y)
        const int lt = tid - 256, G = K >> 3, total = (rpt >> 2) * G;
        const int da = 256 / G, dg = 256 - da * G, af = lt / G, gf = lt - af * G;
        u32x4 v[NU][4];
        int la, lg, wa, wg;                             // the next piece to load, the next to write
        auto step_on = [&](int& a, int& g) {
            a += da; g += dg;
            if (g >= G) { g -= G; a += 1; }
        };
        auto load = [&](int n, const uint16_t* base, int last) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = 4 * la + r < last ? 4 * la + r : last;
                v[n][r] = *reinterpret_cast<const u32x4*>(base + t * ldb + 8 * lg);
            }
            step_on(la, lg);
        };
        auto put = [&](int n) {
            if (lt + 256 * n < total) {
                const u32x4 iv = *reinterpret_cast<const u32x4*>(sInv + 8 * wg);             // 8 positions
                uint8_t* dst = area + 8 * wa;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t pos = (iv[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
                    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
                    const u32x2 w = {__builtin_amdgcn_perm(v[n][1][e >> 1], v[n][0][e >> 1], sel),
                                     __builtin_amdgcn_perm(v[n][3][e >> 1], v[n][2][e >> 1], sel)};
                    *reinterpret_cast<u32x2*>(dst + __umul24(pos, pitch)) = w;
                }
            }
            step_on(wa, wg);
        };
        auto begin = [&]() { la = wa = af; lg = wg = gf; };
        auto source = [&](int t0) { return Bsrc + t0 * ldb; };
        // vmcnt(0): every piece has arrived, also where this thread had none to write (the next loads wait for nothing)
        auto settled = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); };
        constexpr int H = NU / 2;
        int t0 = 0, end = rpt;
        {   // the first tile: written while its second half arrives
            const uint16_t* base = source(0);
            const int last = (end < ntok ? end : ntok) - 1;
            begin();
#pragma unroll
            for (int n = 0; n < H; ++n) load(n, base, last);
            __syncthreads();                             // the inverse permutation is complete
#pragma unroll
            for (int n = H; n < NU; ++n) {
                load(n, base, last);
                put(n - H);
            }
#pragma unroll
            for (int n = NU - H; n < NU; ++n) put(n);
            settled();
        }
        // (a branch around the loads alone would copy their registers where it joins, and wait for them there)
        for (;;) {
            __syncthreads();                             // the tile is complete
            if (end >= ntok) break;
            begin();
            const uint16_t* base = source(end);
            const int last = (ntok - end < rpt ? ntok - end : rpt) - 1;
#pragma unroll
            for (int n = 0; n < NU; ++n) load(n, base, last);            // in flight during this tile's products
            __syncthreads();                             // products done
            __syncthreads();                             // output rows complete
            copy_out(t0, end);
            t0 = end;
            end += rpt;
            __syncthreads();                             // output rows have been read
#pragma unroll
            for (int n = 0; n < NU; ++n) put(n);
            settled();
        }
        __syncthreads();                                 // the last tile: products done
        __syncthreads();                                 // output rows complete
        copy_out(t0, end);
        return;
    }

    // ---- wavefronts 0-3: TM row tiles each against all tokens of the tile
    constexpr int SUB = DENSE ? 2 : 4;                   // sub-steps (32 contraction indices) of a step
    const int l32 = lane & 31, h = lane >> 5;
    const int rt0 = rtb + wave * TM;
    const int nst = DENSE ? 2 * nks : nks;               // steps of 128 (dense: 64) contraction indices, two at least
    const uint8_t* pa[TM];                               // uniform
    const uint8_t* pm[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int rt = rt0 + i < ntr ? rt0 + i : ntr - 1;                // clamped: computed, never stored
        pa[i] = reinterpret_cast<const uint8_t*>(A) + static_cast<int64_t>(rt) * nst * 4096;
        pm[i] = DENSE ? nullptr : reinterpret_cast<const uint8_t*>(Ameta) + static_cast<int64_t>(rt) * nks * 512;
    }
    constexpr int NR = DENSE || TM * TN < 4 ? 2 : 1;     // steps in flight (256 registers)
    u32x4 ra[NR][TM][4];
    u32x2 rm[NR][DENSE ? 1 : TM];
    // the registers of sub-step s4 of step `st` (of slot `u`)
    auto load_meta = [&](int u, int st) {
        uint32_t l8 = lane * 8;
        asm volatile("" : "+v"(l8));
#pragma unroll
        for (int i = 0; i < TM; ++i)
            if constexpr (!DENSE) rm[u][i] = *reinterpret_cast<const u32x2*>(pm[i] + st * 512 + l8);
    };
    auto load_sub = [&](int u, int st, int s4, int i) {
        uint32_t l16 = lane * 16;
        asm volatile("" : "+v"(l16));
#pragma unroll
        for (int x = 0; x < 4 / SUB; ++x)
            ra[u][i][s4 * (4 / SUB) + x] = *reinterpret_cast<const u32x4*>(pa[i] + st * 4096 + (s4 * (4 / SUB) + x) * 1024 + l16);
    };
    clear_tail(tid, 256);
    // lane i of a group of 16 reads column i / 4 of four and tokens 4 (i % 4) .. + 3 of sixteen
    const uint8_t* frag0 = area + (8 * h + ((lane & 15) >> 2)) * pitch + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    const uint8_t* frag[2][2] = {{frag0, frag0 + 4 * pitch}, {frag0 + 64 * pitch, frag0 + 68 * pitch}};
    __syncthreads();                                     // the inverse permutation is complete
    for (int t0 = 0, end = rpt;;) {
        // both slots are requested while the tile is written
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            load_meta(u, u);
#pragma unroll
            for (int s4 = 0; s4 < SUB; ++s4)
#pragma unroll
                for (int i = 0; i < TM; ++i) load_sub(u, u, s4, i);
        }
        f32x16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
        __syncthreads();                                 // the tile is complete
        if (rt0 < ntr) {
            BFragT bf[2][TN];
            // read n of the 4 TN that make up the token fragments of a sub-step
            auto read = [&](int slot, int ofs, int n) {
                bf[slot][n % TN].d[n / TN] = read_turned(frag[n / TN >> 1][n / TN & 1] + ofs + 64 * (n % TN));
            };
            auto first_col = [&](int st) { return DENSE ? (st >> 1) * 128 + (st & 1) * 32 : st * 128; };
            // one step; the registers just used take the same place of the step after the next
            auto step = [&](auto slot_c, int st, auto load_c) {
                constexpr int u = decltype(slot_c)::value;
                constexpr bool LOAD = decltype(load_c)::value;
                u32x2 m[DENSE ? 1 : TM];
                if constexpr (!DENSE) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) m[i] = rm[u][i];
                    if constexpr (LOAD) load_meta(u, st + NR);
                }
#pragma unroll
                for (int s4 = 0; s4 < SUB; ++s4) {
                    int ofs = (s4 + 1 < SUB ? first_col(st) + 16 * (s4 + 1) : first_col(st + 1 < nst ? st + 1 : 0)) * pitch;
                    asm volatile("" : "+s"(ofs));
                    // A wavefront issues in order: fragment reads (a sub-step ahead) and weight loads go between the matrix
                    // instructions, whose execution covers them.
                    constexpr int NX = DENSE ? 2 : 1, NQ = TM * NX * TN, NREAD = 4 * TN;
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
#pragma unroll
                        for (int x = 0; x < NX; ++x) {
#pragma unroll
                            for (int j = 0; j < TN; ++j) {
                                AFragT af;
                                if constexpr (DENSE) {
                                    af.q = ra[u][i][2 * s4 + x];
                                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af.v, bf[s4 & 1][j].half[x], acc[i][j], 0, 0, 0);
                                } else {
                                    af.q = ra[u][i][s4];
                                    const int idx = static_cast<int>(s4 < 2 ? m[i].x : m[i].y);
                                    if (s4 & 1)
                                        acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, bf[s4 & 1][j].v, acc[i][j], idx, 0, 1);
                                    else
                                        acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af.v, bf[s4 & 1][j].v, acc[i][j], idx, 0, 0);
                                }
                                const int q = (i * NX + x) * TN + j;
#pragma unroll
                                for (int n = q * NREAD / NQ; n < (q + 1) * NREAD / NQ; ++n) read((s4 + 1) & 1, ofs, n);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
                        if constexpr (LOAD) load_sub(u, st + NR, s4, i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            using S0 = std::integral_constant<int, 0>;
#pragma unroll
            for (int n = 0; n < 4 * TN; ++n) read(0, 0, n);
            int st = 0;
            if constexpr (NR == 1) {
#pragma unroll 1
                for (; st + 1 < nst; ++st) step(S0{}, st, std::true_type{});
                step(S0{}, st, std::false_type{});
            } else {
                using S1 = std::integral_constant<int, NR - 1>;
#pragma unroll 1
                for (; st + 4 <= nst; st += 2) {
                    step(S0{}, st, std::true_type{});
                    step(S1{}, st + 1, std::true_type{});
                }
                if (!DENSE && nst - st == 3) {
                    step(S0{}, st, std::true_type{});
                    step(S1{}, st + 1, std::false_type{});
                    step(S0{}, st + 2, std::false_type{});
                } else {
                    step(S0{}, st, std::false_type{});
                    step(S1{}, st + 1, std::false_type{});
                }
            }
        }
        __syncthreads();                                 // products done: the area is free
        if (rt0 < ntr) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int t = j * 32 + l32;
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const uint32_t xlo = pack_bf16(acc[i][j][8 * p + 0], acc[i][j][8 * p + 1]);
                        const uint32_t xhi = pack_bf16(acc[i][j][8 * p + 2], acc[i][j][8 * p + 3]);
                        const uint32_t ylo = pack_bf16(acc[i][j][8 * p + 4], acc[i][j][8 * p + 5]);
                        const uint32_t yhi = pack_bf16(acc[i][j][8 * p + 6], acc[i][j][8 * p + 7]);
                        const auto slo = __builtin_amdgcn_permlane32_swap(xlo, ylo, false, false);
                        const auto shi = __builtin_amdgcn_permlane32_swap(xhi, yhi, false, false);
                        const int a0 = (rt0 + i) * 32 + 16 * p + 8 * h;  // first of this lane's 8 weight rows
                        if (t < rpt && a0 + 8 <= Adim) {                 // Adim is a multiple of 8
                            u32x2* d = reinterpret_cast<u32x2*>(area + t * pitchC + 2 * (a0 - a_base));
                            d[0] = (u32x2){slo[0], shi[0]};
                            d[1] = (u32x2){slo[1], shi[1]};
                        }
                    }
                }
        }
        __syncthreads();                                 // output rows complete
        copy_out(t0, end);
        if (end >= ntok) break;
        t0 = end;
        end += rpt;
        __syncthreads();                                 // output rows have been read
        clear_tail(tid, 256);
    }
}

struct ColPlan { int tm, rpt, chunk, rounds; unsigned grid, pieces; size_t lds; };

int col_pitch(int rpt) { return 8 * ((rpt / 4) | 1); }  // an odd number of 8-byte units: columns spread over all banks

size_t col_lds(int rpt, int64_t K, int64_t width) {
    const int64_t rows = round_up(K, 128) * col_pitch(rpt) + 128;        // fragment reads may run past the last column
    const int64_t out = static_cast<int64_t>(rpt) * (2 * width + 8);
    return static_cast<size_t>(round_up(2 * K, 16) + (rows > out ? rows : out));
}

// Row tiles per wavefront, tokens per workgroup and tile.  256 workgroups at most; every one takes the same number of tokens
// in the fewest tiles.  TM by the estimate below: fitted (within 12 %) to 720 timed launches over 136 .. 2048 columns, 32 .. 2600
// rows and 16 .. 60000 tokens; over these its choice costs 0.2 % against the best of the three.  `whole`: all weight rows in one
// workgroup, which then is the only one to read the token rows that it writes (dX on top of dY).
bool col_plan(int64_t Adim, int64_t K, int64_t T, bool dense, bool whole, ColPlan& best) {
    double best_us = 0;
    best.tm = 0;
    for (int tm = 1; tm <= (whole ? 4 : 3); ++tm) {
        const int64_t pieces = ceil_div(Adim, 128 * tm), width = Adim < 128 * tm ? Adim : 128 * tm, slots = 256 / pieces;
        if (slots < 1 || (whole && pieces > 1)) continue;
        int cap = tm == 4 ? 32 : 64;
        while (cap > 0 && (cap * K > 32 * 256 * kColUnits || col_lds(cap, K, width) > kColLds)) cap -= 4;
        if (cap < 4) continue;
        const int64_t chunk = round_up(ceil_div(T, slots), 4), rounds = ceil_div(chunk, cap);
        const int rpt = static_cast<int>(round_up(ceil_div(chunk, rounds), 4)), tn = rpt > 32 ? 2 : 1;
        const int64_t grid = ceil_div(T, chunk);
        const double steps = static_cast<double>(rounds * tm * ceil_div(K, 128)), tokens = static_cast<double>(rounds * rpt * grid * pieces) / 256e4;
        const double us = dense ? 3.26 + 0.15 * rounds + (0.133 + 0.058 * tn) * steps + (0.95 * K + 0.92 * 128 * tm) * tokens
                                : 3.20 + 0.39 * rounds + (0.101 + 0.046 * tn) * steps + (0.86 * K + 0.65 * 128 * tm) * tokens;
        if (best.tm == 0 || us < best_us) {
            best_us = us;
            best = {tm, rpt, static_cast<int>(chunk), static_cast<int>(rounds), static_cast<unsigned>(grid), static_cast<unsigned>(pieces),
                    col_lds(rpt, K, width)};
        }
    }
    return best.tm != 0;
}

// Where this kernel is the faster way.  Narrow outputs: always (2-of-4 and dense; 768 x 40 at 35191 tokens 22.5 -> 21.7 us,
// 1824 x 64 at 18042 54.5 -> 25.9).  Wider ones read every token row once per piece of weight rows, which the other ways do not:
//   2-of-4, beyond 512 terms (else a gathered copy of dY): up to two tiles and 16 pieces (1152 x 1152 at 1087 tokens 15.8 -> 9.1
//   us, 800 x 2368 at 115 7.7 / 7.7) or three pieces (1632 x 736 at 18816 72.7 -> 67.2); 1696 x 1552 at 4570, three tiles of five
//   pieces, 37.0 / 40.9, 2016 x 3360 at 11160 139 / 217.
//   2-of-4, up to 512 terms (else the row-major resident tile): up to two tiles (280 x 1728 at 3504 12.0 -> 11.4), or one
//   piece; 320 x 1088 at 27946 33.8 / 39.5, 384 x 1056 at 16356 20.3 / 24.8.
//   dense (else weights put in natural order): one tile (1376 x 2880 at 2880, two, 56.7 -> 41.9, but 1728 x 896 at 6467 35.9 /
//   43.5), 16 pieces (960 x 2880 at 145, 23 of them, 9.1 / 10.8) and 256 terms.
//   Long contractions in 13 pieces and more, all of which read the tokens: a gathered copy is little next to the weights, and the
//   streaming kernel splits the contraction where its tiles are few.  4:8 from 1320 terms, in pieces of 128 rows from 2.4 million weights and
//   with 29 to 199 tokens (1792 x 1952 at 68 10.4 / 12.8; at 254 1792 x 1712 12.8 / 13.0, at 19 1568 x 1920 10.0 -> 8.9, 1376 x 1600 at 121
//   9.9 -> 8.9), in 14 pieces of 256 up to 512 (1752 x 4056 at 470 21.0 / 24.1, 1632 x 3776 at 527 24.0 -> 21.2); 2:4 from 1920 terms in 14 pieces
//   of 256 (2048 x 3680 at 915 25.6 / 31.8, 1984 x 3808 at 242 14 % faster there; 2016 x 3752 at 515 22.9 -> 19.1).
bool col_gains(const ColPlan& p, int64_t Adim, int64_t K, int64_t T, bool dense) {
    if (Adim <= 512 && Adim <= K) return true;
    if (p.tm == 1 && dense && p.pieces > 12 && K >= 1320 && Adim * K >= 2400000 && T > 28 && T < 200) return false;
    if (p.tm == 2 && p.pieces > 13 && K >= (dense ? 1320 : 1920) && (T <= 512 || (!dense && T > 768))) return false;
    if (dense) return K >= 256 && p.rounds == 1 && p.pieces <= 16;
    return (p.rounds <= 2 && p.pieces <= 16) || p.pieces <= (K > 512 ? 3u : 1u);
}

template <int TM, int TN, bool DENSE, int NU>
int run_coltile(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, const void* Bsrc, int64_t ldb, const int32_t* perm,
                int64_t T, void* C, int64_t ldc, const ColPlan& p, hipStream_t s) {
    auto kern = k_gemm_sp24_coltile<TM, TN, DENSE, NU>;
    static DeviceMemo attr_set;
    const int dev = DeviceMemo::device();
    if (!attr_set.get(dev)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kColLds) != hipSuccess)
            return BIMASK_ERR_HIP;
        attr_set.set(dev, 1);
    }
    const bool stream_out = streams_out(C, Adim, ldc, p.pieces == 1);
    hipLaunchKernelGGL(kern, dim3(p.grid, p.pieces), dim3(kColThreads), p.lds, s, static_cast<const uint16_t*>(A), meta,
                       static_cast<int>(Adim), static_cast<int>(K), static_cast<const uint16_t*>(Bsrc), ldb, perm, T,
                       static_cast<uint16_t*>(C), ldc, p.chunk, p.rpt, col_pitch(p.rpt), stream_out);
    return check_launch();
}

}  // namespace

bool gemm_sp24_coltile_shape(int64_t Adim, int64_t K) { return K > 512 && gemm_dense_coltile_shape(Adim, K); }
bool gemm_dense_coltile_shape(int64_t Adim, int64_t K) {
    return K > 128 && K <= 2048 && K % 8 == 0 && Adim >= 8 && Adim <= 512 && Adim % 8 == 0 && Adim <= K;
}

// Returns BIMASK_ERR_UNSUPPORTED where shape or alignment are outside this kernel, or another one is the faster.
int launch_gemm_sp24_coltile(const void* A, const uint32_t* meta, int64_t Adim, int64_t K, const void* Bsrc, int64_t ldb,
                             const int32_t* perm, int64_t T, void* C, int64_t ldc, hipStream_t s, bool dense) {
    if (!perm || T < 1 || T > 0x7FFFFFFF || K <= 128 || K > 2048 || K % 8 != 0 || Adim < 8 || Adim % 8 != 0) return BIMASK_ERR_UNSUPPORTED;
    if (!aligned16(A) || !aligned16(meta) || !aligned16(Bsrc) || !aligned16(C) || ldb % 8 != 0 || ldc % 8 != 0)
        return BIMASK_ERR_UNSUPPORTED;
    ColPlan p;
    const bool over = !disjoint(Bsrc, T, ldb, K, C, ldc, Adim, 2);
    if (!col_plan(Adim, K, T, dense, over, p) || !col_gains(p, Adim, K, T, dense)) return BIMASK_ERR_UNSUPPORTED;
    const bool few = static_cast<int64_t>(p.rpt) * K <= 32 * 256 * 4;    // pieces per fetching thread
#define BIMASK_CT(TM_, TN_, D_)                                                                                     \
    return few ? run_coltile<TM_, TN_, D_, 4>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p, s)                   \
               : run_coltile<TM_, TN_, D_, kColUnits>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p, s);
#define BIMASK_CT_DENSE(TM_, TN_) { if (dense) BIMASK_CT(TM_, TN_, true) else BIMASK_CT(TM_, TN_, false) }
#define BIMASK_CT_TOKENS(TM_) { if (p.rpt > 32) BIMASK_CT_DENSE(TM_, 2) else BIMASK_CT_DENSE(TM_, 1) }
    switch (p.tm) {
        case 1: BIMASK_CT_TOKENS(1)
        case 2: BIMASK_CT_TOKENS(2)
        case 3: BIMASK_CT_TOKENS(3)
        default:                                                         // 385 .. 512 rows in one piece, 32 tokens
            return dense ? run_coltile<4, 1, true, kColUnits>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p, s)
                         : run_coltile<4, 1, false, kColUnits>(A, meta, Adim, K, Bsrc, ldb, perm, T, C, ldc, p, s);
    }
#undef BIMASK_CT_TOKENS
#undef BIMASK_CT_DENSE
#undef BIMASK_CT
}

}  // namespace bimask
