// Row-permutation search (Sec. 3.3 / Alg. 1 of arXiv 2302.06058): score K candidate
// permutations by their number of eligible N:M column blocks and take the first best.
//
// The forward mask is cut into column slices of 1024 columns (128 bytes per row, one cache
// line; 4096 columns when rows do not start on line boundaries).  A wavefront scores one
// candidate on one slice over a range of row blocks: lane (b, q) = (l / CHL, l % CHL) handles
// row block b of the current step and 16 bytes of the slice, so one load instruction fetches
// whole contiguous row segments through the gather P, and the M rows of a block are added
// bit-sliced (one counter per column, 128 columns per lane at once), compared with N and the
// eligible columns pop-counted.  Workgroups are numbered so that each XCD works on one slice
// at a time: the slice then stays in that XCD's L2 for all K candidates and the mask is read
// from HBM about once.  Partial scores per (slice, row range, candidate) go to scratch; a
// second small kernel sums them, takes the arg-max and copies the winning
// permutation.  Large searches on unaligned masks and groups of many layers score from LDS instead (below).
// Integers only: the result is bit-reproducible.
#include <atomic>

#include "common.hpp"

namespace bimask {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int M> struct Planes { static constexpr int L = M == 4 ? 3 : (M == 8 ? 4 : 5); };

// VEC: rows of the mask start on 16-byte boundaries (whole 16-byte chunks exist or not).
// CHL: 16-byte chunks per row and slice (8 or 32).  U: row-block groups per step, all in
// flight at once.  N2OF4: the 2:4 case, where "more than two of four" is a 7-operation
// boolean formula instead of a bit-sliced adder.
template <int M, bool VEC, int CHL, int U, bool N2OF4>
__device__ __forceinline__ void
perm_score_body(const uint32_t* __restrict__ B_bits, int I, int64_t J, int wpr32,
                const int32_t* __restrict__ perms, int K, int N, int nseg, int sps, int64_t items,
                int32_t* __restrict__ partial, unsigned block, unsigned grid) {
    constexpr int L = Planes<M>::L;
    constexpr int BPS = 64 / CHL;                        // row blocks per load instruction
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // workgroup ids go round-robin over the 8 XCDs: XCD x takes a contiguous range of items
    const int64_t per_xcd = grid / 8;
    const int64_t item = ((block % 8) * per_xcd + block / 8) * (kThreads / 64) + wave;
    if (item >= items) return;
    const int seg = static_cast<int>(item % nseg);
    const int64_t sc = item / nseg;
    const int c = static_cast<int>(sc % K), slice = static_cast<int>(sc / K);
    const int bl = lane / CHL, ch = lane % CHL;
    const int word0 = (slice * CHL + ch) * 4;

    // columns at or beyond J never count; words beyond the row are not read (clamped address)
    uint32_t valid[4];
    int woff[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int64_t nv = J - static_cast<int64_t>(word0 + w) * 32;
        valid[w] = nv >= 32 ? 0xFFFFFFFFu : (nv <= 0 ? 0u : (1u << static_cast<int>(nv)) - 1u);
        woff[w] = word0 + w < wpr32 ? word0 + w : wpr32 - 1;
    }
    const uint32_t* Bs = B_bits + (VEC ? (word0 < wpr32 ? word0 : 0) : 0);

    const int nblk = I / M, steps = (nblk + BPS * U - 1) / (BPS * U);
    const int s_begin = seg * sps;
    const int s_end = s_begin + sps < steps ? s_begin + sps : steps;
    const int32_t* P = perms + static_cast<int64_t>(c) * I;

    int4 pe[U][M / 4];                                   // permutation entries of the next step
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int b = (s_begin * U + u) * BPS + bl;
        b = b < nblk ? b : nblk - 1;                     // clamped: loaded, counted as nothing
#pragma unroll
        for (int v = 0; v < M / 4; ++v) pe[u][v] = *reinterpret_cast<const int4*>(P + static_cast<int64_t>(b) * M + 4 * v);
    }
    int acc = 0;
    for (int s = s_begin; s < s_end; ++s) {
        u32x4 x[U][M];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const int r = (m & 3) == 0 ? pe[u][m >> 2].x : ((m & 3) == 1 ? pe[u][m >> 2].y
                            : ((m & 3) == 2 ? pe[u][m >> 2].z : pe[u][m >> 2].w));
                const uint32_t* row = Bs + static_cast<int64_t>(r) * wpr32;
                if constexpr (VEC) {
                    x[u][m] = *reinterpret_cast<const u32x4*>(row);
                } else {
                    x[u][m].x = row[woff[0]]; x[u][m].y = row[woff[1]]; x[u][m].z = row[woff[2]]; x[u][m].w = row[woff[3]];
                }
            }
        const int sn = s + 1 < s_end ? s + 1 : s;        // the last step reloads its own entries
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int b = (sn * U + u) * BPS + bl;
            b = b < nblk ? b : nblk - 1;
#pragma unroll
            for (int v = 0; v < M / 4; ++v) pe[u][v] = *reinterpret_cast<const int4*>(P + static_cast<int64_t>(b) * M + 4 * v);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int cnt = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t gt;                             // columns whose block holds more than N ones
                if constexpr (N2OF4) {
                    const uint32_t a = x[u][0][w], b = x[u][1][w], cc = x[u][2][w], d = x[u][3][w];
                    gt = (a & b & (cc | d)) | (cc & d & (a | b));
                } else {
                    uint32_t sp[L];
#pragma unroll
                    for (int p = 0; p < L; ++p) sp[p] = 0;
#pragma unroll
                    for (int m = 0; m < M; ++m) {        // bit-sliced add of one bit-row
                        uint32_t carry = x[u][m][w];
#pragma unroll
                        for (int p = 0; p < L; ++p) {
                            const uint32_t t = sp[p] & carry;
                            sp[p] ^= carry;
                            carry = t;
                        }
                    }
                    uint32_t eq = 0xFFFFFFFFu;
                    gt = 0;
#pragma unroll
                    for (int p = L - 1; p >= 0; --p) {
                        if ((N >> p) & 1) { eq &= sp[p]; }
                        else { gt |= eq & sp[p]; eq &= ~sp[p]; }
                    }
                }
                cnt += __popc(~gt & valid[w]);
            }
            acc += (s * U + u) * BPS + bl < nblk ? cnt : 0;   // a clamped (repeated) block counts nothing
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (lane == 0) partial[(static_cast<int64_t>(slice) * nseg + seg) * K + c] = acc;
}

template <int M, bool VEC, int CHL, int U, bool N2OF4>
__global__ void __launch_bounds__(kThreads)
k_perm_score(const uint32_t* __restrict__ B_bits, int I, int64_t J, int wpr32,
             const int32_t* __restrict__ perms, int K, int N, int nseg, int sps, int64_t items,
             int32_t* __restrict__ partial) {
    perm_score_body<M, VEC, CHL, U, N2OF4>(B_bits, I, J, wpr32, perms, K, N, nseg, sps, items, partial, blockIdx.x, gridDim.x);
}

// Grouped launch: the searches of several independent layers in one grid (first[l] = first
// workgroup of layer l, a multiple of 8 so that the XCD assignment of a layer's items holds).
struct ScoreGroupP {
    const uint32_t* B_bits;
    const int32_t* perms;
    int32_t* partial;
    int64_t J, items;
    int I, wpr32, nseg, sps;
};
constexpr int kSearchGroupCap = group_capacity(sizeof(ScoreGroupP));     // 56-byte entries: 63 layers
struct ScoreGroup {
    int n;
    unsigned first[kSearchGroupCap + 1];
    ScoreGroupP p[kSearchGroupCap];
};
template <int M, bool VEC, int CHL, int U, bool N2OF4>
__global__ void __launch_bounds__(kThreads)
k_perm_score_group(const ScoreGroup g, int K, int N) {
    int l = 0;
    while (l + 1 < g.n && blockIdx.x >= g.first[l + 1]) ++l;
    const ScoreGroupP& p = g.p[l];
    perm_score_body<M, VEC, CHL, U, N2OF4>(p.B_bits, p.I, p.J, p.wpr32, p.perms, K, N, p.nseg, p.sps, p.items, p.partial,
                                           blockIdx.x - g.first[l], g.first[l + 1] - g.first[l]);
}

// Sums the per-tile partial scores, takes the first arg-max and copies the winner.
// `piece` of `pieces` workgroups: all of them find the winner (the partial sums are a few KB), each copies its share of
// the permutation, the first one writes the scores.
// A workgroup has 1024 threads: 128 candidates x 8 tile groups at a time, so every
// thread issues its few independent loads at once instead of walking all tiles serially.
constexpr int kFinalThreads = 1024;
__device__ __forceinline__ void
perm_final_body(const int32_t* __restrict__ partial, int ntiles, int K, int64_t I,
                const int32_t* __restrict__ perms, int32_t* __restrict__ scores,
                int32_t* __restrict__ best, int32_t* __restrict__ best_perm, int64_t piece, int64_t pieces) {
    __shared__ int psum[8][128];
    __shared__ long long red[128];
    const int cl = threadIdx.x & 127, part = threadIdx.x >> 7;
    long long mine = -1;
    for (int c0 = 0; c0 < K; c0 += 128) {
        const int c = c0 + cl;
        int s = 0;
        if (c < K) {
            // four independent loads per round: the partial sums are L2 latency, not bandwidth
            int t = part;
            for (; t + 24 < ntiles; t += 32) {
                const int a0 = partial[static_cast<int64_t>(t) * K + c], a1 = partial[static_cast<int64_t>(t + 8) * K + c];
                const int a2 = partial[static_cast<int64_t>(t + 16) * K + c], a3 = partial[static_cast<int64_t>(t + 24) * K + c];
                s += (a0 + a1) + (a2 + a3);
            }
            for (; t < ntiles; t += 8) s += partial[static_cast<int64_t>(t) * K + c];
        }
        psum[part][cl] = s;
        __syncthreads();
        if (part == 0 && c < K) {
            int tot = 0;
#pragma unroll
            for (int p = 0; p < 8; ++p) tot += psum[p][cl];
            if (piece == 0) scores[c] = tot;
            // larger score first, then the smaller candidate index
            const long long key = (static_cast<long long>(tot) << 32) | static_cast<uint32_t>(0x7FFFFFFF - c);
            mine = key > mine ? key : mine;
        }
        __syncthreads();
    }
    if (part == 0) red[cl] = mine;
    __syncthreads();
    for (int off = 64; off > 0; off >>= 1) {
        if (static_cast<int>(threadIdx.x) < off) {
            const long long o = red[threadIdx.x + off];
            if (o > red[threadIdx.x]) red[threadIdx.x] = o;
        }
        __syncthreads();
    }
    const int bc = 0x7FFFFFFF - static_cast<int>(red[0] & 0xFFFFFFFFll);
    if (piece == 0 && threadIdx.x == 0) *best = bc;
    if (best_perm) {
        const int32_t* P = perms + static_cast<int64_t>(bc) * I;
        for (int64_t i = piece * kFinalThreads + threadIdx.x; i < I; i += pieces * kFinalThreads) best_perm[i] = P[i];
    }
}

__global__ void __launch_bounds__(kFinalThreads)
k_perm_final(const int32_t* __restrict__ partial, int ntiles, int K, int64_t I,
             const int32_t* __restrict__ perms, int32_t* __restrict__ scores,
             int32_t* __restrict__ best, int32_t* __restrict__ best_perm) {
    perm_final_body(partial, ntiles, K, I, perms, scores, best, best_perm, blockIdx.x, gridDim.x);
}

struct FinalGroupP {
    const int32_t* partial;
    const int32_t* perms;
    int32_t* scores;
    int32_t* best;
    int32_t* best_perm;
    int64_t I;
    int ntiles;
};
struct FinalGroup {
    FinalGroupP p[kSearchGroupCap];
};
// one workgroup per layer
__global__ void __launch_bounds__(kFinalThreads)
k_perm_final_group(const FinalGroup g, int K) {
    const FinalGroupP& p = g.p[blockIdx.x];
    perm_final_body(p.partial, p.ntiles, K, p.I, p.perms, p.scores, p.best, p.best_perm, 0, 1);
}

// ---- scoring from LDS -------------------------------------------------------------------------------------------
// With K candidates every mask row is read K times, and from L2 that is what the kernel above lives on: 564 MB for
// 4096 x 11008 at K = 100, at 15 TB/s (the rate of its 16-byte gathers) 37 us.  Here a workgroup copies one column slice
// of the mask -- ALL rows, 16 .. 128 bytes of each -- into LDS once and scores a range of candidates on it; L2 only
// delivers the candidates themselves, once per slice.  The widest slice that fits is taken: neighbouring lanes then read
// neighbouring chunks of a row (fewer bank conflicts between random rows), whole cache lines are copied, and the
// candidates are read fewer times.  The slice is zero beyond column J, so that a column outside the matrix never counts
// as "more than N": eligible columns = all columns of the slice - those.  The wavefronts share the (candidate, row-block
// group) pairs of the workgroup evenly; sums meet in LDS (integers: any order).
constexpr int kLdsThreads = 1024;
constexpr int kLdsScoreBytes = 156 * 1024;               // slice; the candidates' sums (kLdsCands) follow
constexpr int kLdsCands = 256;                           // candidates per workgroup at most

// full adder; one three-input bit operation each
__device__ __forceinline__ uint32_t add3(uint32_t a, uint32_t b, uint32_t c) { return a ^ b ^ c; }
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) { return (a & b) | (c & (a | b)); }

// bit planes of the number of ones among 8 words
__device__ __forceinline__ void planes8(const uint32_t* x, uint32_t (&p)[4]) {
    const uint32_t s0 = add3(x[0], x[1], x[2]), c0 = maj3(x[0], x[1], x[2]);
    const uint32_t s1 = add3(x[3], x[4], x[5]), c1 = maj3(x[3], x[4], x[5]);
    const uint32_t s2 = add3(s0, s1, x[6]), c2 = maj3(s0, s1, x[6]);
    const uint32_t c3 = s2 & x[7];
    const uint32_t t = add3(c0, c1, c2), d = maj3(c0, c1, c2);
    p[0] = s2 ^ x[7];
    p[1] = t ^ c3;
    p[2] = d ^ (t & c3);
    p[3] = d & t & c3;
}

// columns (bits) whose M rows hold more than N ones
template <int M, bool N2OF4>
__device__ __forceinline__ uint32_t more_than_n(const uint32_t (&x)[M], int N) {
    if constexpr (N2OF4) return (maj3(x[0], x[1], x[2]) & x[3]) | (x[0] & x[1] & x[2]);
    uint32_t sp[Planes<M>::L];
    if constexpr (M == 4) {
        const uint32_t s0 = add3(x[0], x[1], x[2]), c0 = maj3(x[0], x[1], x[2]), c1 = s0 & x[3];
        sp[0] = s0 ^ x[3]; sp[1] = c0 ^ c1; sp[2] = c0 & c1;
    } else if constexpr (M == 8) {
        planes8(x, sp);
    } else {
        uint32_t a[4], b[4];
        planes8(x, a);
        planes8(x + 8, b);
        uint32_t carry = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) { sp[p] = add3(a[p], b[p], carry); carry = maj3(a[p], b[p], carry); }
        sp[4] = carry;
    }
    uint32_t eq = 0xFFFFFFFFu, gt = 0;
#pragma unroll
    for (int p = Planes<M>::L - 1; p >= 0; --p) {
        if ((N >> p) & 1) { eq &= sp[p]; }
        else { gt |= eq & sp[p]; eq &= ~sp[p]; }
    }
    return gt;
}

// One layer's share: `block` = slice * groups + group; the group takes the candidates [group * cpg, ...).
// sh: log2 of the 16-byte chunks per row of the slice.
struct ScoreLdsP {
    const uint32_t* B_bits;
    const int32_t* perms;
    int32_t* partial;
    int64_t J;
    int I, wpr32, sh, groups, cpg;
};
template <int M, bool N2OF4>
__device__ __forceinline__ void perm_score_lds_body(const ScoreLdsP& p, int K, int N, int block) {
    extern __shared__ u32x4 slice_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sh = p.sh, chl = 1 << sh, I = p.I;
    const int slice = block / p.groups, c0 = (block - slice * p.groups) * p.cpg;
    const int nc = p.cpg < K - c0 ? p.cpg : K - c0;
    if (nc <= 0) return;                                 // whole workgroup
    int* sum = reinterpret_cast<int*>(slice_lds + (static_cast<int64_t>(I) << sh));
    const int wslice = slice * 4 * chl;                  // first mask word of the slice
    const int64_t cols_left = p.J - static_cast<int64_t>(wslice) * 32;
    const int ncols = static_cast<int>(cols_left < 128 * chl ? cols_left : 128 * chl);

    // copy the slice: whole chunks of aligned rows as 16-byte loads, eight in flight per thread
    const bool vec = p.wpr32 % 4 == 0 && (reinterpret_cast<uintptr_t>(p.B_bits) & 15u) == 0;
    const int total = I << sh;
    for (int q0 = tid; q0 < total; q0 += 8 * kLdsThreads) {
        u32x4 v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int q = q0 + e * kLdsThreads;
            v[e] = (u32x4){0u, 0u, 0u, 0u};
            if (q < total) {
                const int w0 = wslice + 4 * (q & (chl - 1));
                const uint32_t* src = p.B_bits + static_cast<int64_t>(q >> sh) * p.wpr32 + w0;
                if (vec) {
                    if (w0 < p.wpr32) v[e] = *reinterpret_cast<const u32x4*>(src);
                } else {
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        if (w0 + w < p.wpr32) v[e][w] = src[w];
                }
                const int left = ncols - 128 * (q & (chl - 1));          // columns of this chunk that exist
                if (left < 128) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const int n = left - 32 * w;
                        v[e][w] &= n >= 32 ? 0xFFFFFFFFu : (n <= 0 ? 0u : (1u << n) - 1u);
                    }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (q0 + e * kLdsThreads < total) slice_lds[q0 + e * kLdsThreads] = v[e];
    }
    for (int c = tid; c < nc; c += kLdsThreads) sum[c] = 0;
    __syncthreads();

    // A wavefront walks over groups of D steps of one candidate each (64 >> sh row blocks a step); the candidate's entries
    // for the next group are requested before this group is counted.
    constexpr int D = M == 16 ? 2 : 4;
    const int nblk = I / M, bps = 64 >> sh, groups = (nblk + D * bps - 1) / (D * bps);
    const int all = nc * groups, per = (all + kLdsThreads / 64 - 1) / (kLdsThreads / 64);
    int it = wave * per;
    const int end = it + per < all ? it + per : all;
    if (it < end) {
        const int bl = lane >> sh;
        const char* mine = reinterpret_cast<const char*>(slice_lds + (lane & (chl - 1)));
        int c = it / groups, g = it - c * groups;
        auto fetch = [&](int4 (&pe)[D][M / 4], int cc, int gg) {
            const char* src = reinterpret_cast<const char*>(p.perms + static_cast<int64_t>(c0 + cc) * I);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                int b = (gg * D + d) * bps + bl;
                b = b < nblk ? b : nblk - 1;             // clamped: read, counted as nothing
#pragma unroll
                for (int v = 0; v < M / 4; ++v) pe[d][v] = *reinterpret_cast<const int4*>(src + static_cast<uint32_t>(b) * (4 * M) + 16 * v);
            }
        };
        int4 pe[D][M / 4];
        fetch(pe, c, g);
        int acc = 0;
        for (; it < end; ++it) {
            int4 cur[D][M / 4];
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int v = 0; v < M / 4; ++v) cur[d][v] = pe[d][v];
            const bool last = g + 1 == groups;           // of this candidate
            const int cn = last ? (c + 1 < nc ? c + 1 : c) : c, gn = last ? 0 : g + 1;
            fetch(pe, cn, gn);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                u32x4 x[M];
#pragma unroll
                for (int v = 0; v < M / 4; ++v) {
                    x[4 * v + 0] = *reinterpret_cast<const u32x4*>(mine + (static_cast<uint32_t>(cur[d][v].x) << (sh + 4)));
                    x[4 * v + 1] = *reinterpret_cast<const u32x4*>(mine + (static_cast<uint32_t>(cur[d][v].y) << (sh + 4)));
                    x[4 * v + 2] = *reinterpret_cast<const u32x4*>(mine + (static_cast<uint32_t>(cur[d][v].z) << (sh + 4)));
                    x[4 * v + 3] = *reinterpret_cast<const u32x4*>(mine + (static_cast<uint32_t>(cur[d][v].w) << (sh + 4)));
                }
                int cnt = 0;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    uint32_t xw[M];
#pragma unroll
                    for (int m = 0; m < M; ++m) xw[m] = x[m][w];
                    cnt += __popc(more_than_n<M, N2OF4>(xw, N));
                }
                acc += (g * D + d) * bps + bl < nblk ? cnt : 0;
            }
            if (last || it + 1 == end) {                 // wave-uniform: this candidate's sum leaves the registers
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
                if (lane == 0) atomicAdd(&sum[c], acc);
                acc = 0;
            }
            c = last ? c + 1 : c;
            g = gn;
        }
    }
    __syncthreads();
    for (int i = tid; i < nc; i += kLdsThreads)
        p.partial[static_cast<int64_t>(slice) * K + c0 + i] = ncols * nblk - sum[i];
}

template <int M, bool N2OF4>
__global__ void __launch_bounds__(kLdsThreads)
k_perm_score_lds(const ScoreLdsP p, int K, int N) { perm_score_lds_body<M, N2OF4>(p, K, N, static_cast<int>(blockIdx.x)); }

constexpr int kLdsGroupCap = group_capacity(sizeof(ScoreLdsP));
struct ScoreLdsGroup {
    int n;
    unsigned first[kLdsGroupCap + 1];
    ScoreLdsP p[kLdsGroupCap];
};
template <int M, bool N2OF4>
__global__ void __launch_bounds__(kLdsThreads)
k_perm_score_lds_group(const ScoreLdsGroup g, int K, int N) {
    int l = 0;
    while (l + 1 < g.n && blockIdx.x >= g.first[l + 1]) ++l;
    perm_score_lds_body<M, N2OF4>(g.p[l], K, N, static_cast<int>(blockIdx.x - g.first[l]));
}

struct LdsPlan {
    int sh, nslices, steps;                              // steps of one candidate on one slice
    size_t lds;
};
// A slice takes up to `slice_bytes`.  false: the search takes the L2 kernel (few candidates, which do not pay for the copy;
// more rows than LDS holds at 16 bytes each; or more slices than the scratch has room for).
bool plan_lds(int64_t I, int64_t J, int K, int M, size_t ws_bytes, int64_t slice_bytes, LdsPlan& pl) {
    if (K < 16 || I * 16 > kLdsScoreBytes) return false;
    int sh = 3;
    while (sh > 0 && ((I << sh) * 16 > slice_bytes || (128ll << (sh - 1)) >= J)) --sh;
    if (sh == 0 && J > 128) return false;                // 16 bytes of every line: the copy costs too much
    pl.sh = sh;
    pl.nslices = static_cast<int>(ceil_div(J, 128ll << sh));
    pl.steps = static_cast<int>(round_up(ceil_div(I / M, 64 >> sh), M == 16 ? 2 : 4));
    pl.lds = (static_cast<size_t>(I) << sh) * 16 + kLdsCands * sizeof(int32_t);
    return static_cast<size_t>(pl.nslices) * static_cast<size_t>(K) * sizeof(int32_t) <= ws_bytes;
}
// candidates of one slice cut into groups of `cpg`
void cut_candidates(int K, int64_t groups, int& ngroups, int& cpg) {
    const int64_t most = ceil_div(K, 4), least = ceil_div(K, kLdsCands);
    groups = groups > most ? most : groups;
    groups = groups < least ? least : groups;
    cpg = static_cast<int>(ceil_div(K, groups));
    ngroups = static_cast<int>(ceil_div(K, cpg));
}
// What either kernel takes, in us: sums of a few counts with measured rates (per ratio: the counting of 2:4 is a formula, that
// of 16 rows an adder tree of planes).  Alone, over 390 searches from 128 x 128 to 9984 x 20000 with 16 .. 400 candidates,
// the estimates stray by 7-11 %.
int ratio_class(int N, int M) { return M == 4 ? (N == 2 ? 0 : 1) : (M == 8 ? 2 : 3); }
// 16-byte loads of the L2 kernel per lane: M rows per row block, four 4-byte loads where rows start inside 16 bytes
double l2_loads(int64_t I, int64_t J, int K, int M, const PermPlan& pl) {
    const int64_t blocks = round_up(ceil_div(I / M, 64 / pl.chunks), M == 16 ? 1 : 2);
    return static_cast<double>(blocks) * pl.nslices * K * M * (ceil_div(J, 32) % 4 ? 4 : 1);
}
// steps of the busiest of a workgroup's 16 wavefronts
int64_t lds_steps(int cpg, int steps, int M) {
    const int d = M == 16 ? 2 : 4;
    return ceil_div(static_cast<int64_t>(cpg) * (steps / d), kLdsThreads / 64) * d;
}
// A layer alone.  Where mask rows are whole cache lines the L2 kernel reaches 22-24 TB/s and the copy does not pay
// (4096 x 4096 at K = 100 14.5 us from L2, 15.0 from LDS); where rows start inside lines every gather touches two, and
// large searches gain: 4096 x 11008 37.8 -> 25.9 us, 4096 x 2304 17.2 -> 13.2, while 2048 x 2304 takes 11.3 / 11.2,
// 1024 x 4608 10.3 / 10.9 and 4096 x 2304 with 32 candidates 9.6 / 11.1.  Rows that are not 16-byte aligned, read word by
// word from L2, gain earlier (3072 x 1504 20.4 -> 13.7).  Other ratios count longer on the same bytes: 4:8 2048 x 4608 at
// K = 100 18.3 -> 14.2, but 1024 x 11008 15.2 / 17.7 and 4096 x 11008 at 32 candidates 18.6 / 22.9: they compare estimates.
bool alone_from_lds(int64_t I, int64_t J, int N, int M, int K, const PermPlan& pl, const LdsPlan& lp) {
    const int64_t words = ceil_div(J, 32);
    if (words % 32 == 0 || K < 32 || I * J < (words % 4 ? 300000000 : 600000000) / K) return false;
    if (M == 4 && N == 2) return true;
    static constexpr struct { double base, step, copy16, copy4, l2_base; } kCost[3] = {      // us; per step, per byte copied by a workgroup
        {4.6, .725, 2.7e-5, 5.3e-5, 6.8}, {2.1, 1.43, 4.8e-5, 7.2e-5, 7.8}, {2.2, 3.1, 5.1e-5, 7.4e-5, 8.7}};
    const auto& c = kCost[ratio_class(N, M) - 1];
    int ngroups, cpg;
    cut_candidates(K, 256 / lp.nslices, ngroups, cpg);
    const double rounds = static_cast<double>(ceil_div(static_cast<int64_t>(lp.nslices) * ngroups, 256));
    const double lds = c.base + rounds * (c.step * lds_steps(cpg, lp.steps, M)
                                          + (words % 4 ? c.copy4 : c.copy16) * static_cast<double>((I << lp.sh) * 16));
    return lds < .97 * (c.l2_base + 53e-6 * l2_loads(I, J, K, M, pl));
}

template <typename Kern>
bool allow_lds(Kern kern, DeviceMemo& memo) {
    const int dev = DeviceMemo::device();
    if (memo.get(dev)) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            kLdsScoreBytes + kLdsCands * static_cast<int>(sizeof(int32_t))) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    memo.set(dev, 1);
    return true;
}
// May the kernels take their LDS?  Where the runtime refuses, the search stays with the L2 kernel.
template <int M, bool N2OF4>
bool lds_allowed() {
    static DeviceMemo memo;
    return allow_lds(k_perm_score_lds<M, N2OF4>, memo);
}
template <int M, bool N2OF4>
bool lds_group_allowed() {
    static DeviceMemo memo;
    return allow_lds(k_perm_score_lds_group<M, N2OF4>, memo);
}
template <int M>
bool lds_group_allowed(int N) { return M == 4 && N == 2 ? lds_group_allowed<M, M == 4>() : lds_group_allowed<M, false>(); }

// BIMASK_ERR_UNSUPPORTED: left to the L2 kernel
template <int M, bool N2OF4>
int run_score_lds(const uint32_t* B_bits, int64_t I, int64_t J, int N, const int32_t* perms, int K, const LdsPlan& pl,
                  int32_t* partial, hipStream_t s) {
    if (!lds_allowed<M, N2OF4>()) return BIMASK_ERR_UNSUPPORTED;
    ScoreLdsP p{B_bits, perms, partial, J, static_cast<int>(I), static_cast<int>(ceil_div(J, 32)), pl.sh, 1, K};
    cut_candidates(K, 256 / pl.nslices, p.groups, p.cpg);        // one workgroup per CU, one round where that is possible
    hipLaunchKernelGGL((k_perm_score_lds<M, N2OF4>), dim3(static_cast<unsigned>(pl.nslices * p.groups)), dim3(kLdsThreads), pl.lds, s,
                       p, K, N);
    return check_launch();
}

template <int M>
int run_score(const uint32_t* B_bits, int64_t I, int64_t J, int N, const int32_t* perms, int K,
              const PermPlan& pl, int32_t* partial, int& ntiles, hipStream_t s) {
    constexpr int U = M == 16 ? 1 : 2;
    LdsPlan lp;
    if (plan_lds(I, J, K, M, pl.ws_bytes, kLdsScoreBytes, lp) && alone_from_lds(I, J, N, M, K, pl, lp)) {
        const int rc = M == 4 && N == 2 ? run_score_lds<M, M == 4>(B_bits, I, J, N, perms, K, lp, partial, s)
                                        : run_score_lds<M, false>(B_bits, I, J, N, perms, K, lp, partial, s);
        if (rc != BIMASK_ERR_UNSUPPORTED) {
            ntiles = lp.nslices;
            return rc;
        }
    }
    ntiles = pl.ntiles;
    const int wpr32 = static_cast<int>(ceil_div(J, 32));
    const int64_t items = static_cast<int64_t>(pl.ntiles) * K;
    const unsigned grid = static_cast<unsigned>(round_up(ceil_div(items, kThreads / 64), 8));
    const bool vec = aligned16(B_bits) && wpr32 % 4 == 0;
#define BIMASK_SCORE(VEC, CHL)                                                                               \
    {                                                                                                        \
        if (M == 4 && N == 2)                                                                                \
            hipLaunchKernelGGL((k_perm_score<M, VEC, CHL, U, M == 4>), dim3(grid), dim3(kThreads), 0, s, B_bits, \
                               static_cast<int>(I), J, wpr32, perms, K, N, pl.nseg, pl.sps, items, partial); \
        else                                                                                                 \
            hipLaunchKernelGGL((k_perm_score<M, VEC, CHL, U, false>), dim3(grid), dim3(kThreads), 0, s, B_bits, \
                               static_cast<int>(I), J, wpr32, perms, K, N, pl.nseg, pl.sps, items, partial); \
    }
    if (pl.chunks == 32) { if (vec) BIMASK_SCORE(true, 32) else BIMASK_SCORE(false, 32) }
    else                 { if (vec) BIMASK_SCORE(true, 8)  else BIMASK_SCORE(false, 8) }
#undef BIMASK_SCORE
    return check_launch();
}

}  // namespace

PermPlan plan_perm_search(int64_t I, int64_t J, int K, int M) {
    PermPlan pl{};
    const int64_t pitch = ceil_div(J, 32) * 4;                   // bytes per mask row
    pl.chunks = (pitch % 128 != 0 && J >= 4096) ? 32 : 8;
    pl.nslices = static_cast<int>(ceil_div(J, pl.chunks * 128));
    const int U = M == 16 ? 1 : 2;
    const int64_t steps = ceil_div(I / M, (64 / pl.chunks) * U); // row blocks per wavefront step
    // about 32 wavefronts per CU, at least 2 steps each
    int64_t nseg = ceil_div(8192, static_cast<int64_t>(pl.nslices) * K);
    const int64_t nseg_max = steps / 2 > 1 ? steps / 2 : 1;
    nseg = nseg < 1 ? 1 : (nseg > nseg_max ? nseg_max : nseg);
    pl.sps = static_cast<int>(ceil_div(steps, nseg));
    pl.nseg = static_cast<int>(ceil_div(steps, pl.sps));
    pl.ntiles = pl.nslices * pl.nseg;
    pl.ws_bytes = static_cast<size_t>(pl.ntiles) * K * sizeof(int32_t);
    return pl;
}

namespace {

// score kernels of the layers that share one instantiation (row alignment, slice width)
template <int M>
int run_score_group(const bimask_group_layer* L, const int* which, int cnt, int N, int K, bool vec, int chunks,
                    hipStream_t s) {
    constexpr int U = M == 16 ? 1 : 2;
    ScoreGroup g{};
    g.n = cnt;
    unsigned blocks = 0;
    for (int l = 0; l < cnt; ++l) {
        const bimask_group_layer& a = L[which[l]];
        const PermPlan pl = plan_perm_search(a.I, a.J, K, M);
        ScoreGroupP& p = g.p[l];
        p.B_bits = a.B_bits; p.perms = a.perms; p.partial = static_cast<int32_t*>(a.workspace);
        p.J = a.J; p.I = static_cast<int>(a.I);
        p.wpr32 = static_cast<int>(ceil_div(a.J, 32));
        p.nseg = pl.nseg; p.sps = pl.sps;
        p.items = static_cast<int64_t>(pl.ntiles) * K;
        g.first[l] = blocks;
        blocks += static_cast<unsigned>(round_up(ceil_div(p.items, kThreads / 64), 8));
    }
    g.first[cnt] = blocks;
#define BIMASK_SCOREG(VEC, CHL)                                                                              \
    {                                                                                                        \
        if (M == 4 && N == 2)                                                                                \
            hipLaunchKernelGGL((k_perm_score_group<M, VEC, CHL, U, M == 4>), dim3(blocks), dim3(kThreads), 0, s, g, K, N); \
        else                                                                                                 \
            hipLaunchKernelGGL((k_perm_score_group<M, VEC, CHL, U, false>), dim3(blocks), dim3(kThreads), 0, s, g, K, N);  \
    }
    if (chunks == 32) { if (vec) BIMASK_SCOREG(true, 32) else BIMASK_SCOREG(false, 32) }
    else              { if (vec) BIMASK_SCOREG(true, 8)  else BIMASK_SCOREG(false, 8) }
#undef BIMASK_SCOREG
    return check_launch();
}

// Layers of one group call.  The L2 kernel cuts every layer into thousands of wavefronts and the fixed costs of these add
// up over the layers, with a launch per alignment of the rows; the LDS launch costs its copies and at least 7-13 us, and
// ratios other than 2:4 count longer.  So the two are compared by what they would take, in us, with rates fitted to 290 groups of 2 ..
// 63 layers (the estimates stray by 7-17 %); the LDS launch has to be the shorter one by 5 %.  2:4, 100 candidates: 54 ResNet-50
// matrices 45 -> 23 us, 48 transformer matrices 41 -> 23 (with 16 candidates 12.8 / 15.3), 63 of 64 x 64 14.5 / 15.2; 4:8, 100
// candidates: 48 transformer matrices 46 -> 40, 36 of 1152 x 9216 244 / 306.
constexpr int kGroupFromLds = 32;                        // layers: below, all from L2
struct GroupCost {
    double base, layer, worst, total, copy;              // LDS: per layer; per step of the longest workgroup / of all; per byte
    double l2_base, l2_class, l2_wave, l2_load16, l2_load4, l2_line;     // L2: per launch after the first, wavefront, load, line
};
constexpr GroupCost kGroupCost[4] = {
    {7.2, .09, .115, 1.03e-3, 1.76e-7, 6.5, 3.4, 4.4e-4, 8.6e-6, 17.3e-6, 1.75e-6},
    {8.2, .07, .257, 2.18e-3, 1.63e-7, 6.3, 4.0, 3.8e-4, 3.7e-6, 13.6e-6, 5.33e-6},
    {13.5, .02, .080, 4.96e-3, 1.63e-7, 7.0, 5.3, 6.0e-4, 24.4e-6, 16.2e-6, 2.25e-6},
    {10.6, .05, 1.65, 7.86e-3, 1.07e-7, 7.3, 5.0, 7.1e-4, 25.1e-6, 14.9e-6, 2.20e-6}};

// equal shares, a bit under one workgroup per CU over the layers together (54 ResNet-50 matrices at K = 100: 21 us
// with 192 shares, 23-24 with 128, 256 or 384), none below two groups of steps per wavefront
int64_t lds_share(const LdsPlan* plans, int cnt, int K) {
    int64_t all = 0;
    for (int l = 0; l < cnt; ++l) all += static_cast<int64_t>(plans[l].nslices) * K * plans[l].steps;
    return all / 192 > 128 ? all / 192 : 128;
}
// which class of the L2 launches a layer belongs to: (rows 16-byte aligned?, 8 or 32 chunks per slice)
int l2_class(const bimask_group_layer& a, int K, int M) {
    return (aligned16(a.B_bits) && ceil_div(a.J, 32) % 4 == 0 ? 1 : 0) | (plan_perm_search(a.I, a.J, K, M).chunks == 32 ? 2 : 0);
}
// others: bit set of the classes that stay with the L2 kernel whatever is decided here
bool group_from_lds(const bimask_group_layer* L, const int* which, const LdsPlan* plans, int cnt, int N, int M, int K, unsigned others) {
    if (cnt < kGroupFromLds) return false;
    const GroupCost& c = kGroupCost[ratio_class(N, M)];
    const int64_t share = lds_share(plans, cnt, K);
    int64_t worst = 0;
    double total = 0, copy = 0, l2 = c.l2_base - c.l2_class;
    unsigned classes = others;
    for (int l = 0; l < cnt; ++l) {
        const bimask_group_layer& a = L[which[l]];
        int ngroups, cpg;
        cut_candidates(K, ceil_div(static_cast<int64_t>(K) * plans[l].steps, share), ngroups, cpg);
        const int64_t steps = lds_steps(cpg, plans[l].steps, M), wgs = static_cast<int64_t>(plans[l].nslices) * ngroups;
        worst = steps > worst ? steps : worst;
        total += static_cast<double>(steps) * wgs;
        copy += static_cast<double>((a.I << plans[l].sh) * 16) * wgs;
        const PermPlan pl = plan_perm_search(a.I, a.J, K, M);
        const int64_t words = ceil_div(a.J, 32);
        const int cls = l2_class(a, K, M);
        if (!((classes >> cls) & 1u)) l2 += c.l2_class;
        classes |= 1u << cls;
        l2 += c.l2_wave * pl.ntiles * K + (words % 4 ? c.l2_load4 : c.l2_load16) * l2_loads(a.I, a.J, K, M, pl)
            + c.l2_line * static_cast<double>(a.I * K * (ceil_div(words, 32) + (words % 32 ? 1 : 0)));
    }
    const double lds = c.base + c.layer * cnt + c.worst * worst + c.total * total + c.copy * copy;
    return lds < .95 * l2;
}

// All layers that score from LDS, in one launch whatever the alignment of their rows (two workgroups per CU: half of LDS
// each where a layer allows it).
template <int M>
int run_score_lds_group(const bimask_group_layer* L, const int* which, const LdsPlan* plans, int cnt, int N, int K, hipStream_t s) {
    static_assert(kLdsGroupCap >= kSearchGroupCap && sizeof(ScoreLdsGroup) <= 3840, "argument tables must fit the kernel arguments");
    ScoreLdsGroup g{};
    g.n = cnt;
    const int64_t share = lds_share(plans, cnt, K);
    size_t lds = 0;
    unsigned blocks = 0;
    for (int l = 0; l < cnt; ++l) {
        const bimask_group_layer& a = L[which[l]];
        ScoreLdsP& p = g.p[l];
        p = ScoreLdsP{a.B_bits, a.perms, static_cast<int32_t*>(a.workspace), a.J, static_cast<int>(a.I),
                      static_cast<int>(ceil_div(a.J, 32)), plans[l].sh, 1, K};
        cut_candidates(K, ceil_div(static_cast<int64_t>(K) * plans[l].steps, share), p.groups, p.cpg);
        g.first[l] = blocks;
        blocks += static_cast<unsigned>(plans[l].nslices * p.groups);
        lds = plans[l].lds > lds ? plans[l].lds : lds;
    }
    g.first[cnt] = blocks;
    if (M == 4 && N == 2) hipLaunchKernelGGL((k_perm_score_lds_group<M, M == 4>), dim3(blocks), dim3(kLdsThreads), lds, s, g, K, N);
    else hipLaunchKernelGGL((k_perm_score_lds_group<M, false>), dim3(blocks), dim3(kLdsThreads), lds, s, g, K, N);
    return check_launch();
}

}  // namespace

// The searches of n independent layers (same N:M and number of candidates) in a few launches:
// one scoring launch per kernel instantiation in use, one finalising launch with a workgroup
// per layer.  Same results as n calls of launch_perm_search.
int launch_perm_search_group(const bimask_group_layer* L, int n, int N, int M, int K, hipStream_t s) {
    static_assert(sizeof(FinalGroup) <= 3840 && sizeof(ScoreGroup) <= 3840, "argument tables must fit the kernel arguments");
    for (int b = 0; b < n; b += kSearchGroupCap) {
        const int m = n - b < kSearchGroupCap ? n - b : kSearchGroupCap;
        int ntiles[kSearchGroupCap], from_lds[kSearchGroupCap], nl = 0;
        unsigned others = 0;
        LdsPlan plans[kSearchGroupCap];
        for (int l = 0; l < m; ++l) {
            const bimask_group_layer& a = L[b + l];
            const PermPlan pl = plan_perm_search(a.I, a.J, K, M);
            ntiles[l] = pl.ntiles;
            if (plan_lds(a.I, a.J, K, M, pl.ws_bytes, kLdsScoreBytes / 2, plans[nl])) from_lds[nl++] = b + l;
            else others |= 1u << l2_class(a, K, M);
        }
        if (!group_from_lds(L, from_lds, plans, nl, N, M, K, others)
            || !(M == 4 ? lds_group_allowed<4>(N) : M == 8 ? lds_group_allowed<8>(N) : lds_group_allowed<16>(N))) nl = 0;
        for (int l = 0; l < nl; ++l) ntiles[from_lds[l] - b] = plans[l].nslices;
        if (nl) {
            int rc = BIMASK_ERR_NM;
            if (M == 4) rc = run_score_lds_group<4>(L, from_lds, plans, nl, N, K, s);
            else if (M == 8) rc = run_score_lds_group<8>(L, from_lds, plans, nl, N, K, s);
            else if (M == 16) rc = run_score_lds_group<16>(L, from_lds, plans, nl, N, K, s);
            if (rc != BIMASK_OK) return rc;
        }
        for (int cls = 0; cls < 4; ++cls) {              // (rows 16-byte aligned?, 8 or 32 chunks per slice)
            const bool vec = cls & 1;
            const int chunks = (cls & 2) ? 32 : 8;
            int which[kSearchGroupCap], cnt = 0;
            for (int l = 0, skip = 0; l < m; ++l) {
                if (skip < nl && from_lds[skip] == b + l) { ++skip; continue; }
                const bimask_group_layer& a = L[b + l];
                if (l2_class(a, K, M) == cls) which[cnt++] = b + l;
            }
            if (cnt == 0) continue;
            int rc = BIMASK_ERR_NM;
            if (M == 4) rc = run_score_group<4>(L, which, cnt, N, K, vec, chunks, s);
            else if (M == 8) rc = run_score_group<8>(L, which, cnt, N, K, vec, chunks, s);
            else if (M == 16) rc = run_score_group<16>(L, which, cnt, N, K, vec, chunks, s);
            if (rc != BIMASK_OK) return rc;
        }
        FinalGroup f{};
        for (int l = 0; l < m; ++l) {
            const bimask_group_layer& a = L[b + l];
            FinalGroupP& p = f.p[l];
            p.partial = static_cast<const int32_t*>(a.workspace); p.perms = a.perms; p.scores = a.scores; p.best = a.best;
            p.best_perm = a.best_perm; p.I = a.I;
            p.ntiles = ntiles[l];
        }
        hipLaunchKernelGGL(k_perm_final_group, dim3(static_cast<unsigned>(m)), dim3(kFinalThreads), 0, s, f, K);
        if (int rc = check_launch()) return rc;
    }
    return BIMASK_OK;
}

int launch_perm_search(const uint32_t* B_bits, int64_t I, int64_t J, int N, int M, const int32_t* perms, int K,
                       int32_t* scores, int32_t* best, int32_t* best_perm, void* ws, hipStream_t s) {
    const PermPlan pl = plan_perm_search(I, J, K, M);
    int32_t* partial = static_cast<int32_t*>(ws);
    int rc = BIMASK_ERR_NM, ntiles = 0;
    if (M == 4) rc = run_score<4>(B_bits, I, J, N, perms, K, pl, partial, ntiles, s);
    else if (M == 8) rc = run_score<8>(B_bits, I, J, N, perms, K, pl, partial, ntiles, s);
    else if (M == 16) rc = run_score<16>(B_bits, I, J, N, perms, K, pl, partial, ntiles, s);
    if (rc != BIMASK_OK) return rc;
    // long permutations are copied by several workgroups (11008 rows: the whole search 32.1 -> 30.8 us)
    const unsigned pieces = best_perm && I > 2 * kFinalThreads ? static_cast<unsigned>(I / (2 * kFinalThreads) < 16 ? I / (2 * kFinalThreads) : 16) : 1u;
    hipLaunchKernelGGL(k_perm_final, dim3(pieces), dim3(kFinalThreads), 0, s, partial, ntiles, K, I, perms, scores, best,
                       best_perm);
    return check_launch();
}

// ---- the search for callers that cannot allocate: partial scores in a static device array --------
// One copy of the array exists per GPU the library runs on, for the life of the process.  In host
// code the array's name is only a handle for hipGetSymbolAddress: the address the kernels get is
// looked up once per device, with that device current, and remembered.
constexpr size_t kStaticScratchBytes = BIMASK_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t perm_search_static_capacity() { return kStaticScratchBytes; }

int launch_perm_search_static(const uint32_t* B_bits, int64_t I, int64_t J, int N, int M, const int32_t* perms, int K,
                              int32_t* scores, int32_t* best, int32_t* best_perm, hipStream_t s) {
    static std::atomic<void*> device_ptr[kMaxDevices];       // zero-initialised: not looked up yet
    if (plan_perm_search(I, J, K, M).ws_bytes > kStaticScratchBytes) return BIMASK_ERR_WORKSPACE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BIMASK_ERR_HIP;
    void* ptr = device_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return BIMASK_ERR_HIP;
        }
        device_ptr[dev].store(ptr, std::memory_order_release);
    }
    // every partial score the second kernel reads is written by the first: nothing to clear
    return launch_perm_search(B_bits, I, J, N, M, perms, K, scores, best, best_perm, ptr, s);
}

namespace {

// Debug helper: is every candidate a permutation of 0 .. I-1?  One workgroup per candidate marks the
// values it meets in an LDS bitmap; a value out of range or met twice clears the candidate's flag.
__global__ void __launch_bounds__(kThreads)
k_check_perms(const int32_t* __restrict__ perms, int64_t I, int32_t* __restrict__ ok) {
    extern __shared__ uint32_t seen[];
    const int words = static_cast<int>((I + 31) >> 5);
    for (int w = threadIdx.x; w < words; w += kThreads) seen[w] = 0u;
    __syncthreads();
    const int32_t* P = perms + static_cast<int64_t>(blockIdx.x) * I;
    int bad = 0;
    for (int64_t r = threadIdx.x; r < I; r += kThreads) {
        const int32_t v = P[r];
        if (v < 0 || v >= I) {
            bad = 1;
        } else {
            const uint32_t bit = 1u << (v & 31);
            if (atomicOr(&seen[v >> 5], bit) & bit) bad = 1;
        }
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) ok[blockIdx.x] = bad ? 0 : 1;
}

}  // namespace

int launch_check_perms(const int32_t* perms, int K, int64_t I, int32_t* ok, hipStream_t s) {
    static DeviceMemo attr_set;
    if (I > kCheckPermsMaxRows) return BIMASK_ERR_UNSUPPORTED;
    const size_t lds = static_cast<size_t>((I + 31) >> 5) * 4;
    const int dev = DeviceMemo::device();
    if (lds > 48 * 1024 && !attr_set.get(dev)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(k_check_perms), hipFuncAttributeMaxDynamicSharedMemorySize,
                                128 * 1024) != hipSuccess) {
            (void)hipGetLastError();
            return BIMASK_ERR_HIP;
        }
        attr_set.set(dev, 1);
    }
    hipLaunchKernelGGL(k_check_perms, dim3(static_cast<unsigned>(K)), dim3(kThreads), lds, s, perms, I, ok);
    return check_launch();
}

}  // namespace bimask
