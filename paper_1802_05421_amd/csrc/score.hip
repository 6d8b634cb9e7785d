// Node anomaly scores (Algorithm 4 with the CAD edge score of the Background
// section), without materialising any n x n commute-time matrix.
//
//   build_zhat  Zh = [sqrt(vol0) Z0 | sqrt(vol1) Z1] over the common nodes
//               (each half padded to 16 columns), sq_c = |Zh0_c|^2 - |Zh1_c|^2
//   score       G = Zh0 Zh0^T - Zh1 Zh1^T on FP64 MFMA over tiles covering
//               the upper triangle (one pass over k, the sums negated half
//               way); per pair a < b, dc_ab = sq_a + sq_b - 2 G_ab
//               = c_0(a,b) - c_1(a,b) (eq. 1 in embedding form), weighted by
//               |W1 - W0| on request; |dc| is summed per row into one
//               partial per (column block, node) and per column into one
//               partial per (row block, node)
//   reduce      F_a = sum of exactly the written partials (fixed order)
//   topk        the best K of every chunk in order, repeated on the candidates
//               (order: value desc, index asc)
//   edges       the K largest edge scores (a < b) exactly: maxima per 256 x 128
//               tile from k_score, threshold = K-th largest tile maximum, only
//               tiles reaching it recomputed and their edges collected
#include <algorithm>
#include <vector>

#include "batch.h"
#include "caddelag.h"
#include "common.h"
#include "gemm.h"
#include "kernels.h"

namespace cdl {

int64_t score_ldz(int64_t k) { return 2 * ((k + 15) / 16 * 16); }

// Row c of the signature embeddings (one wave).
__device__ inline void build_zhat_row(const double *Z0, const double *Z1, const int32_t *map0,
                                      const int32_t *map1, int64_t m, int64_t k, int64_t ldz,
                                      const double *stats0, const double *stats1, double *Zh,
                                      double *sq, int64_t c) {
    const int lane = threadIdx.x;
    const double s0 = sqrt(stats0[0]), s1 = sqrt(stats1[0]);
    double acc = 0.0;
    int64_t a = -1, b = -1;
    if (c < m) {
        a = map0 ? map0[c] : c;
        b = map1 ? map1[c] : c;
    }
    for (int64_t r = lane; r < ldz / 2; r += 64) {
        double x0 = 0.0, x1 = 0.0;
        if (c < m && r < k) {
            x0 = s0 * Z0[a * k + r];
            x1 = s1 * Z1[b * k + r];
        }
        Zh[c * ldz + r] = x0;
        Zh[c * ldz + ldz / 2 + r] = x1;
        acc += x0 * x0 - x1 * x1;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) sq[c] = acc;
}

// One wave per common node; tmax != nullptr: also clears the ntiles tile
// maxima to -1 (no edge).
__global__ void k_build_zhat(const double *Z0, const double *Z1, const int32_t *map0,
                             const int32_t *map1, int64_t m, int64_t k, int64_t ldz,
                             const double *stats0, const double *stats1, double *Zh, double *sq,
                             double *tmax, int64_t ntiles) {
    build_zhat_row(Z0, Z1, map0, map1, m, k, ldz, stats0, stats1, Zh, sq, blockIdx.x);
    if (tmax)
        for (int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x; i < ntiles; i += (int64_t)gridDim.x * 64)
            tmax[i] = -1.0;
}

hipError_t launch_build_zhat(const double *Z0, const double *Z1, const int32_t *map0,
                             const int32_t *map1, int64_t m, int64_t mpad, int64_t k,
                             const double *stats0, const double *stats1, double *Zh, double *sq,
                             double *tmax, hipStream_t s) {
    hipLaunchKernelGGL(k_build_zhat, dim3((unsigned)mpad), dim3(64), 0, s, Z0, Z1, map0, map1,
                       m, k, score_ldz(k), stats0, stats1, Zh, sq, tmax,
                       (int64_t)rect_upper_tiles(mpad));
    return hipGetLastError();
}

// Tile shapes of the score Gram (the same edge scores from each).  0: 256 x
// 128 in bands of four row blocks; 1 and 2: square tiles, two or three
// workgroups on a CU; 3: as 2 with 64-bit addresses, for very many columns.  Only pairs a < b count: a tile straddling the diagonal
// also holds pairs a > b, whose mirror images another element covers.
constexpr int kScoreFar = 3;
static_assert(kScoreFar + 1 == kScoreShapes, "score shapes");
template <int SHAPE> struct ScoreCfg {
    static constexpr int WM = SHAPE == 0 ? 4 : 2, WN = SHAPE == 1 ? 4 : 2;
    static constexpr int TM = SHAPE == 0 ? 256 : SHAPE == 1 ? 128 : 64, TN = SHAPE >= 2 ? 64 : 128;
    // waves per SIMD that the registers must leave room for: one, two and
    // three workgroups on a CU
    static constexpr int WAVES = SHAPE == 0 ? 2 : SHAPE == 1 ? 4 : 3;
    using Core = Dma64Core<TM, TN, WM, WN, SHAPE >= 2 ? 3 : 2, SHAPE == kScoreFar>;
};
__host__ __device__ static int64_t score_tm(int shape) { return shape == 0 ? 256 : shape == 1 ? 128 : 64; }
__host__ __device__ static int64_t score_tn(int shape) { return shape >= 2 ? 64 : 128; }

int score_tile_count(int shape, int64_t mpad) {
    if (shape == 0) return rect_upper_tiles(mpad);
    const int nt = (int)(mpad / score_tn(shape));
    return nt * (nt + 1) / 2;
}

// Doubles of partial sums that a shape writes: one slot of mpad entries per
// column block and one per row block.
static int64_t score_part_need(int shape, int64_t mpad) {
    return (mpad / score_tm(shape) + mpad / score_tn(shape)) * mpad;
}

int64_t score_part_doubles(int64_t mpad, int64_t kpad) {
    return (mpad / 128 + mpad / 256 + 2 * kpad) * mpad;
}

// The shape whose busiest CU has the least work, over one pair or the pairs of
// a group, among those whose partial sums fit every pair's workspace.  A 64 x
// 64 tile loses about a tenth of the matrix pipes' rate to its shorter
// k-tiles (0.90 against 1.86-1.89 ms' worth at 256 x 128 and 128 x 128 on
// large products); on 20 to 600 large tiles the last round of CUs costs more
// than that.  Weighted scores are bound by the gathers of the weights as well,
// which only the 64 x 64 tiles keep in flight (a tenth more for the others).
// From 2^20 columns on the rows of a 256-row tile take 2^32 bytes, which the
// first three shapes' offsets do not.
int score_shape(int P, const int64_t *mpad, int64_t kpad, int weighted) {
    if (score_ldz(kpad) >= (int64_t)1 << 21) return kScoreFar;
    int best = 0;
    double tb = 1e300;
    for (int q = 0; q < kScoreFar; ++q) {
        if (weighted && q == 1) continue;
        int64_t tiles = 0;
        bool fits = true;
        for (int t = 0; t < P; ++t) {
            tiles += score_tile_count(q, mpad[t]);
            fits = fits && score_part_need(q, mpad[t]) <= score_part_doubles(mpad[t], kpad);
        }
        const double t = (double)cdiv(tiles, 256) * (double)(score_tm(q) * score_tn(q)) / (q == 2 && !weighted ? 0.90 : 1.0);
        if (fits && t < tb) { tb = t; best = q; }
    }
    return best;
}

// Edge score omega_ab |c_0(a,b) - c_1(a,b)| of common nodes a != b from the
// signature Gram entry G_ab and, weighted, the two weights (shared by the node
// and the edge kernels, so both see bit-identical values).
__device__ inline double edge_score(double G, double sqa, double sqb, int weighted, double w0,
                                    double w1) {
    double v = fabs(sqa + sqb - 2.0 * G);
    if (weighted) v *= fabs(w1 - w0);
    return v;
}

// Partial sums: row a's sum over the columns of tile (I, J) goes to
// part[J][a], column b's sum over the rows of the tile to part[ncol + I][b];
// each slot has exactly one writer.  tmax != nullptr: also fold the tile's
// largest edge score over a < b into the maximum of its 256 x 128 tile.
template <int SHAPE> struct ScoreShared {
    using Cfg = ScoreCfg<SHAPE>;
    double srow[Cfg::WN][Cfg::TM], scol[Cfg::WM][Cfg::TN], smax[Cfg::WM * Cfg::WN];
};

// Upper-triangle tile `id` of the score Gram with its partial sums (one
// workgroup).  Bound by the FP64 matrix pipes: 2 m^2 k flop.  The square
// shapes put two (three) workgroups on a CU, so that one's sums, weight
// gathers and first loads run under another's MFMAs; with one 256 x 128 tile
// per CU nothing did.
template <int SHAPE, bool WT>
__device__ __forceinline__ void score_tile(const double *Zh, int64_t ldz,
                                  const double *sq, int64_t m, int64_t mpad, const double *W0,
                                  int64_t ld0, const double *W1, int64_t ld1,
                                  const int32_t *map0, const int32_t *map1,
                                  double *part, double *tmax, int id, char *smem_raw,
                                  ScoreShared<SHAPE> &sh) {
    using Cfg = ScoreCfg<SHAPE>;
    using Core = typename Cfg::Core;
    constexpr int WM = Cfg::WM, WN = Cfg::WN, TM = Cfg::TM, TN = Cfg::TN;
    double *smem = (double *)smem_raw;
    auto &srow = sh.srow;
    auto &scol = sh.scol;
    auto &smax = sh.smax;
    const int ncol = (int)(mpad / TN);
    int I, J;
    if (SHAPE == 0) upper_band_tile<4>(id, 0, ncol / 2, ncol, I, J);
    else sym_tile<8>(id, ncol, I, J);
    const int64_t m0 = (int64_t)I * TM, n0 = (int64_t)J * TN;
    Core g;
    g.template run<true>(Zh, ldz, Zh, ldz, m0, n0, ldz, smem);   // Zh1 Zh1^T - Zh0 Zh0^T

    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int wm = wid % WM, wn = wid / WM;
    double cs[Core::WTN], vmax = -1.0, sqb[Core::WTN];
    int64_t j0[Core::WTN], j1[Core::WTN];   // this lane's columns in W0 and W1
#pragma unroll
    for (int b = 0; b < Core::WTN; ++b) {
        cs[b] = 0.0;
        const int64_t gb = n0 + Core::col_of(b), c = gb < m ? gb : m - 1;
        sqb[b] = sq[gb];
        j0[b] = WT && map0 ? map0[c] : c;
        j1[b] = WT && map1 ? map1[c] : c;
    }
    constexpr bool PRE = WT && SHAPE >= 2;   // (the larger shapes have no registers for it)
#pragma unroll
    for (int a = 0; a < Core::WTM; ++a) {
        // the weights of four rows, all loads in flight (indices clamped into
        // the common nodes, so that no load waits behind a test: 166 us a
        // launch at m = 5003, k = 128 against 233 with a load per test)
        double w0[MfmaF64::R][Core::WTN], w1[MfmaF64::R][Core::WTN];
        if (PRE) {
            int64_t i0[MfmaF64::R], i1[MfmaF64::R];
#pragma unroll
            for (int rr = 0; rr < MfmaF64::R; ++rr) {
                const int64_t ga = m0 + Core::row_of(a, rr), c = ga < m ? ga : m - 1;
                i0[rr] = map0 ? map0[c] : c;
                i1[rr] = map1 ? map1[c] : c;
            }
#pragma unroll
            for (int rr = 0; rr < MfmaF64::R; ++rr)
#pragma unroll
                for (int b = 0; b < Core::WTN; ++b) {
                    w0[rr][b] = W0[i0[rr] * ld0 + j0[b]];
                    w1[rr][b] = W1[i1[rr] * ld1 + j1[b]];
                }
        }
#pragma unroll
        for (int rr = 0; rr < MfmaF64::R; ++rr) {
            const int lr = Core::row_of(a, rr);
            const int64_t ga = m0 + lr;
            const double sqa = sq[ga];
            double rs = 0.0;
#pragma unroll
            for (int b = 0; b < Core::WTN; ++b) {
                const int64_t gb = n0 + Core::col_of(b);
                double v = 0.0;
                if (ga < gb && gb < m) {
                    // a branch, not a select: hoisted together, the lane masks of
                    // the selects spill the scalar registers
                    asm volatile("");
                    double x0 = 0.0, x1 = 0.0;
                    if (PRE) {
                        x0 = w0[rr][b];
                        x1 = w1[rr][b];
                    } else if (WT) {
                        x0 = W0[(map0 ? map0[ga] : ga) * ld0 + j0[b]];
                        x1 = W1[(map1 ? map1[ga] : ga) * ld1 + j1[b]];
                    }
                    v = edge_score(-g.acc[a][b][rr], sqa, sqb[b], WT, x0, x1);
                    vmax = fmax(vmax, v);
                }
                rs += v;
                cs[b] += v;
            }
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) rs += __shfl_xor(rs, off);
            if ((lane & 15) == 0) srow[wn][lr] = rs;
        }
    }
#pragma unroll
    for (int b = 0; b < Core::WTN; ++b) {
        double v = cs[b];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        if (lane < 16) scol[wm][Core::col_of(b)] = v;
    }
    if (tmax) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) vmax = fmax(vmax, __shfl_xor(vmax, o));
        if (lane == 0) smax[wid] = vmax;
    }
    __syncthreads();
    if (tmax && threadIdx.x == 0) {
        double mx = smax[0];
        for (int q = 1; q < Core::NT / 64; ++q) mx = fmax(mx, smax[q]);
        // maxima are -1 or >= 0: their bit patterns order like signed integers
        const int cell = SHAPE == 0 ? id : upper_band_id<4>((int)(m0 / 256), (int)(n0 / 128), (int)(mpad / 128));
        atomicMax((long long *)tmax + cell, (long long)__double_as_longlong(mx));
    }
    for (int t = threadIdx.x; t < TM; t += Core::NT) {
        double rs = 0.0;
#pragma unroll
        for (int q = 0; q < WN; ++q) rs += srow[q][t];
        part[(int64_t)J * mpad + m0 + t] = rs;
    }
    for (int t = threadIdx.x; t < TN; t += Core::NT) {
        double cs2 = 0.0;
#pragma unroll
        for (int q = 0; q < WM; ++q) cs2 += scol[q][t];
        part[(int64_t)(ncol + I) * mpad + n0 + t] = cs2;
    }
}

template <int SHAPE, bool WT>
__global__ __launch_bounds__(ScoreCfg<SHAPE>::Core::NT, ScoreCfg<SHAPE>::WAVES) void k_score(
    const double *Zh, int64_t ldz, const double *sq, int64_t m, int64_t mpad, const double *W0,
    int64_t ld0, const double *W1, int64_t ld1, const int32_t *map0, const int32_t *map1,
    double *part, double *tmax, int total) {
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    __shared__ ScoreShared<SHAPE> sh;
    const int w = grid_row_id();
    if (w >= total) return;
    score_tile<SHAPE, WT>(Zh, ldz, sq, m, mpad, W0, ld0, W1, ld1, map0, map1, part, tmax,
                          xcd_remap(w, total), smem_raw, sh);
}

template <int SHAPE, bool WT>
static hipError_t score_launch(const double *Zh, int64_t ldz, const double *sq, int64_t m,
                               int64_t mpad, const double *W0, int64_t ld0, const double *W1,
                               int64_t ld1, const int32_t *map0, const int32_t *map1,
                               double *part, double *tmax, hipStream_t s) {
    using Core = typename ScoreCfg<SHAPE>::Core;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void *)k_score<SHAPE, WT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)Core::SMEM);
        if (e != hipSuccess) return e;
        attr = true;
    }
    const int total = score_tile_count(SHAPE, mpad);
    hipLaunchKernelGGL((k_score<SHAPE, WT>), grid_rows(total), dim3(Core::NT), Core::SMEM, s, Zh, ldz, sq,
                       m, mpad, W0, ld0, W1, ld1, map0, map1, part, tmax, total);
    return hipGetLastError();
}

hipError_t launch_score(int shape, const double *Zh, int64_t k, const double *sq,
                        int64_t m, int64_t mpad, const double *W0, int64_t ld0,
                        const double *W1, int64_t ld1, const int32_t *map0,
                        const int32_t *map1, int weighted, double *part, double *tmax,
                        hipStream_t s) {
    const int64_t ldz = score_ldz(k);
    switch (2 * shape + (weighted ? 1 : 0)) {
#define CDL_CASE(q, w) \
    case 2 * q + w: return score_launch<q, w>(Zh, ldz, sq, m, mpad, W0, ld0, W1, ld1, map0, map1, part, tmax, s);
    CDL_CASE(0, 0) CDL_CASE(0, 1) CDL_CASE(1, 0) CDL_CASE(2, 0) CDL_CASE(2, 1) CDL_CASE(3, 0) CDL_CASE(3, 1)
#undef CDL_CASE
    default: return hipErrorInvalidValue;
    }
}

int score_tiles_2d(int64_t mpad) { return rect_upper_tiles(mpad); }

// ---------------------------------------------------------------------------
// Top edges.  The K largest maxima of the 256 x 128 tiles are K distinct
// edges, so the K-th largest edge score is at least tau = the K-th largest
// tile maximum (when there are fewer than K tiles, tau = -1 and every edge is
// collected).  Only tiles whose maximum reaches tau are recomputed (same core,
// same epilogue arithmetic as k_score); their edges a < b with score >= tau are
// appended to the candidate list.

__global__ void k_edge_threshold(const double *tmax, const int32_t *tile_order, int K,
                                 int ntiles, double *tau, unsigned int *count) {
    if (threadIdx.x != 0) return;
    *tau = ntiles >= K ? tmax[tile_order[K - 1]] : -1.0;
    *count = 0;
}

// Workgroup w: 64 x 64 part w % 8 of tile w / 8 (a reached tile's eight parts
// on eight CUs: about K tiles are reached, so whole tiles left most of the
// chip idle: 85 us with the threshold kernel against 43 at m = 9216, k = 128).
template <int SHAPE>
__global__ __launch_bounds__(ScoreCfg<SHAPE>::Core::NT) void k_edge_collect(
    const double *Zh, int64_t ldz, const double *sq, int64_t m,
    const double *W0, int64_t ld0, const double *W1, int64_t ld1, const int32_t *map0,
    const int32_t *map1, int weighted, int64_t mpad, const double *tmax,
    const double *tau, int64_t cap, unsigned int *count, double *cval, int64_t *cidx) {
    using Core = typename ScoreCfg<SHAPE>::Core;
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    double *smem = (double *)smem_raw;
    const int w = grid_row_id(), id = w >> 3, sub = w & 7, ncol = (int)(mpad / 128);
    if (id >= rect_upper_tiles(mpad)) return;
    const double th = *tau;
    if (tmax[id] < th) return;   // uniform over the workgroup
    int I, J;
    upper_band_tile<4>(id, 0, ncol / 2, ncol, I, J);
    const int64_t m0 = (int64_t)I * 256 + 64 * (sub >> 1), n0 = (int64_t)J * 128 + 64 * (sub & 1);
    if (m0 > n0) return;         // no pair a < b
    Core g;
    g.template run<true>(Zh, ldz, Zh, ldz, m0, n0, ldz, smem);
#pragma unroll
    for (int a = 0; a < Core::WTM; ++a)
#pragma unroll
        for (int rr = 0; rr < MfmaF64::R; ++rr) {
            const int64_t ga = m0 + Core::row_of(a, rr);
#pragma unroll
            for (int b = 0; b < Core::WTN; ++b) {
                const int64_t gb = n0 + Core::col_of(b);
                if (ga < m && gb < m && ga < gb) {
                    double w0 = 0.0, w1 = 0.0;
                    if (weighted) {
                        w0 = W0[(map0 ? map0[ga] : ga) * ld0 + (map0 ? map0[gb] : gb)];
                        w1 = W1[(map1 ? map1[ga] : ga) * ld1 + (map1 ? map1[gb] : gb)];
                    }
                    const double v = edge_score(-g.acc[a][b][rr], sq[ga], sq[gb], weighted, w0, w1);
                    if (v >= th) {
                        const unsigned int q = atomicAdd(count, 1u);
                        if ((int64_t)q < cap) {
                            cval[q] = v;
                            cidx[q] = ga * m + gb;
                        }
                    }
                }
            }
        }
}

template <int SHAPE>
static hipError_t edge_collect_launch(const double *Zh, int64_t ldz, const double *sq, int64_t m,
                                      int64_t mpad, const double *W0, int64_t ld0, const double *W1,
                                      int64_t ld1, const int32_t *map0, const int32_t *map1,
                                      int weighted, const double *tmax, const double *tau, int64_t cap,
                                      unsigned int *count, double *cval, int64_t *cidx, hipStream_t s) {
    using Core = typename ScoreCfg<SHAPE>::Core;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void *)k_edge_collect<SHAPE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)Core::SMEM);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL(k_edge_collect<SHAPE>, grid_rows((int64_t)rect_upper_tiles(mpad) * 8), dim3(Core::NT),
                       Core::SMEM, s, Zh, ldz, sq, m, W0, ld0, W1, ld1, map0, map1, weighted, mpad,
                       tmax, tau, cap, count, cval, cidx);
    return hipGetLastError();
}

hipError_t launch_edge_collect(int shape, const double *Zh, int64_t k,
                               const double *sq, int64_t m, int64_t mpad, const double *W0,
                               int64_t ld0, const double *W1, int64_t ld1,
                               const int32_t *map0, const int32_t *map1, int weighted,
                               const double *tmax, const int32_t *tile_order, int K,
                               double *tau, int64_t cap, unsigned int *count, double *cval,
                               int64_t *cidx, hipStream_t s) {
    hipLaunchKernelGGL(k_edge_threshold, dim3(1), dim3(64), 0, s, tmax, tile_order, K,
                       rect_upper_tiles(mpad), tau, count);
    if (shape == kScoreFar)
        return edge_collect_launch<kScoreFar>(Zh, score_ldz(k), sq, m, mpad, W0, ld0, W1, ld1, map0, map1,
                                              weighted, tmax, tau, cap, count, cval, cidx, s);
    return edge_collect_launch<2>(Zh, score_ldz(k), sq, m, mpad, W0, ld0, W1, ld1, map0, map1, weighted,
                                  tmax, tau, cap, count, cval, cidx, s);
}

// flag = 1 if some entry of map0 lies outside [0, n0) or of map1 outside
// [0, n1), else 0.  One workgroup; the flag needs no initial value.
__global__ __launch_bounds__(1024) void k_check_maps(const int32_t *map0, const int32_t *map1,
                                                     int64_t m, int64_t n0, int64_t n1,
                                                     int *flag) {
    int bad = 0;
#pragma unroll 8
    for (int64_t c = threadIdx.x; c < m; c += 1024) {
        const int32_t a = map0[c], b = map1[c];
        bad |= (a < 0 || a >= n0 || b < 0 || b >= n1);
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) *flag = bad ? 1 : 0;
}

hipError_t launch_check_maps(const int32_t *map0, const int32_t *map1, int64_t m, int64_t n0,
                             int64_t n1, int *flag, hipStream_t s) {
    hipLaunchKernelGGL(k_check_maps, dim3(1), dim3(1024), 0, s, map0, map1, m, n0, n1, flag);
    return hipGetLastError();
}

// F_a = its row partials over the column blocks from its row block's diagonal
// on, then its column partials over the row blocks down to its column block:
// exactly the slots the score tiles (tm x tn) wrote, summed in a fixed order: of
// more than 8 column blocks every fourth slot in a chain of its own, so that the 80
// of 5003 nodes in small tiles do not round one sum 80 times (error against 64 bits
// 1.2e-16 of the scores, one chain 2.6e-16; 256 x 128 tiles in one chain 1.7e-16).
__device__ inline void score_reduce_node(const double *part, int64_t tm, int64_t tn, int64_t m,
                                         int64_t mpad, double *F, int64_t a) {
    if (a >= m) return;
    const int ncol = (int)(mpad / tn), J0 = (int)(a / tm * (tm / tn));
    const int Imax = (int)(a / tn * tn / tm);
    const double *const rows = part + (int64_t)J0 * mpad + a, *const cols = part + (int64_t)ncol * mpad + a;
    if (ncol <= 8) {
        double f = 0.0;
        for (int q = 0; q < ncol - J0; ++q) f += rows[q * mpad];
        for (int q = 0; q <= Imax; ++q) f += cols[q * mpad];
        F[a] = f;
        return;
    }
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    quarter_sums(rows, mpad, ncol - J0, s);
    quarter_sums(cols, mpad, Imax + 1, s);
    F[a] = (s[0] + s[1]) + (s[2] + s[3]);
}

__global__ void k_score_reduce(const double *part, int64_t tm, int64_t tn, int64_t m, int64_t mpad,
                               double *F) {
    score_reduce_node(part, tm, tn, m, mpad, F, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

hipError_t launch_score_reduce(int shape, const double *part, int64_t m, int64_t mpad, double *F,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_score_reduce, dim3((unsigned)cdiv(m, 64)), dim3(64), 0, s, part,
                       score_tm(shape), score_tn(shape), m, mpad, F);
    return hipGetLastError();
}

// ---- grouped over the pairs of a sequence ------------------------------------

__global__ void k_build_zhat_grouped(const BatchPair *pairs, const int *prefix, int P, int64_t k,
                                     int64_t ldz) {
    const int p = group_find(prefix, P, blockIdx.x);
    const BatchPair &q = pairs[p];
    build_zhat_row(q.Z0, q.Z1, q.map0, q.map1, q.m, k, ldz, q.stats0, q.stats1, q.Zh, q.sq,
                   blockIdx.x - prefix[p]);
}

template <int SHAPE, bool WT>
__global__ __launch_bounds__(ScoreCfg<SHAPE>::Core::NT, ScoreCfg<SHAPE>::WAVES) void k_score_grouped(
    const BatchPair *pairs, const int *prefix, int P, int64_t ldz) {
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    __shared__ ScoreShared<SHAPE> sh;
    const int p = group_find(prefix, P, blockIdx.x);
    const BatchPair &q = pairs[p];
    const int id = xcd_remap(blockIdx.x - prefix[p], prefix[p + 1] - prefix[p]);
    score_tile<SHAPE, WT>(q.Zh, ldz, q.sq, q.m, q.mpad, q.W0, q.ld0, q.W1, q.ld1, q.map0, q.map1,
                          q.part, nullptr, id, smem_raw, sh);
}

__global__ void k_score_reduce_grouped(const BatchPair *pairs, const int *prefix, int P) {
    const int p = group_find(prefix, P, blockIdx.x);
    const BatchPair &q = pairs[p];
    score_reduce_node(q.part, score_tm(q.shape), score_tn(q.shape), q.m, q.mpad, q.F,
                      (int64_t)(blockIdx.x - prefix[p]) * blockDim.x + threadIdx.x);
}

template <int SHAPE, bool WT>
static hipError_t score_grouped_launch(const BatchPair *pairs, const int *prefix, int total, int P,
                                       int64_t ldz, hipStream_t s) {
    using Core = typename ScoreCfg<SHAPE>::Core;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void *)k_score_grouped<SHAPE, WT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)Core::SMEM);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL((k_score_grouped<SHAPE, WT>), dim3(total), dim3(Core::NT), Core::SMEM, s, pairs,
                       prefix, P, ldz);
    return hipGetLastError();
}

hipError_t launch_score_grouped(const BatchPair *pairs, const int *prefix_zhat,
                                int total_zhat, const int *prefix_score, int pitch,
                                const int *total_score, const int *prefix_red, int total_red, int P,
                                int64_t k, int weighted, hipStream_t s) {
    const int64_t ldz = score_ldz(k);
    hipLaunchKernelGGL(k_build_zhat_grouped, dim3(total_zhat), dim3(64), 0, s, pairs, prefix_zhat, P,
                       k, ldz);
    hipError_t e = hipGetLastError();
    for (int shape = 0; shape < kScoreShapes && e == hipSuccess; ++shape) {
        const int total = total_score[shape], *prefix = prefix_score + (size_t)shape * pitch;
        if (total == 0) continue;
        switch (2 * shape + (weighted ? 1 : 0)) {
#define CDL_CASE(q, w) \
        case 2 * q + w: e = score_grouped_launch<q, w>(pairs, prefix, total, P, ldz, s); break;
        CDL_CASE(0, 0) CDL_CASE(0, 1) CDL_CASE(1, 0) CDL_CASE(2, 0) CDL_CASE(2, 1) CDL_CASE(3, 0) CDL_CASE(3, 1)
#undef CDL_CASE
        default: return hipErrorInvalidValue;
        }
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_score_reduce_grouped, dim3(total_red), dim3(64), 0, s, pairs, prefix_red, P);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Top-K of (value, index) pairs by descending value, ascending index.

// Chunks of 512 (one pair per thread): twice the largest K, so every round at
// least halves the candidates, and small enough that the first round spreads
// over many workgroups.  What bounds a round is the latency of a chain of
// dependent steps: each wave sorts its 64 pairs by lane shuffles (21 steps), then
// every pair finds its place in the seven other waves' runs by binary searches
// side by side (7 steps).  A whole bitonic sort of the chunk (45 steps, six of
// them through LDS with a barrier) took 11.3 us a launch, this 8.9.
constexpr int kChunk = 512;
static_assert(kChunk >= 2 * CDL_MAX_TOPK, "every round must shrink the candidates");

template <typename I> struct TopkShared {
    unsigned long long key[kChunk];
    I i[kChunk];
};

__device__ inline int32_t shfl_xor_idx(int32_t x, int o) { return __shfl_xor(x, o); }
__device__ inline int64_t shfl_xor_idx(int64_t x, int o) { return __shfl_xor((long long)x, o); }

// Keys in the order of the values (both zeros alike; a NaN of either sign before
// all numbers, so that no pair is lost behind the padding).
__device__ inline unsigned long long topk_key(double v) {
    unsigned long long u = (unsigned long long)__double_as_longlong(v + 0.0);
    if (v != v) u &= 0x7fffffffffffffffull;
    return u >> 63 ? ~u : u | 0x8000000000000000ull;
}

// Place of thread t's pair among the chunk's (512 threads): descending value,
// ascending index, then the padding's copies by wave.
template <typename I> __device__ inline int topk_place(unsigned long long &key, I &i, TopkShared<I> &sh) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
#pragma unroll
    for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const unsigned long long ok = __shfl_xor(key, stride);
            const I oi = shfl_xor_idx(i, stride);
            const bool ahead = ok > key || (ok == key && oi < i);   // the partner comes first
            const bool behind = ok < key || (ok == key && oi > i);
            if (((lane & stride) == 0) == ((lane & size) == 0) ? ahead : behind) {
                key = ok;
                i = oi;
            }
        }
    }
    sh.key[t] = key;
    sh.i[t] = i;
    __syncthreads();
    // pairs of run r before this one; of equal padding, that of the earlier waves
    auto before = [&](int r, int q) {
        const unsigned long long k = sh.key[64 * r + q];
        const I x = sh.i[64 * r + q];
        return k > key || (k == key && (x < i || (x == i && r < wv)));
    };
    int pos[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) pos[r] = 0;
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1)
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (before(r, pos[r] + step - 1)) pos[r] += step;
    int place = lane;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (before(r, pos[r])) ++pos[r];   // (the last of the run)
        place += r == wv ? 0 : pos[r];
    }
    return place;
}

// Chunk b of (val, idx) pairs (idx_in == nullptr: the position); its K best
// to val_out / idx_out + b K.
template <typename I>
__device__ inline void topk_chunk(const double *val_in, const I *idx_in, int64_t count, int K,
                                  double *val_out, I *idx_out, int64_t b, TopkShared<I> &sh) {
    const int64_t p = b * kChunk + threadIdx.x;
    double v = -INFINITY;
    I i = sizeof(I) == 4 ? (I)0x7fffffff : (I)INT64_MAX;
    if (p < count) {
        v = val_in[p];
        i = idx_in ? idx_in[p] : (I)p;
    }
    unsigned long long key = topk_key(v);
    const int place = topk_place(key, i, sh);
    if (place < K) {
        if (val_out)
            val_out[b * K + place] =
                __longlong_as_double((long long)(key >> 63 ? key & 0x7fffffffffffffffull : ~key));
        idx_out[b * K + place] = i;
    }
}

template <typename I>
__global__ __launch_bounds__(kChunk) void k_topk(const double *val_in, const I *idx_in, int64_t count,
                                                 int K, double *val_out, I *idx_out) {
    __shared__ TopkShared<I> sh;
    topk_chunk<I>(val_in, idx_in, count, K, val_out, idx_out, blockIdx.x, sh);
}

int64_t topk_scratch_elems(int64_t m, int K) { return cdiv(m, kChunk) * (int64_t)K; }

// Rounds of k_topk on `count` pairs (none: one round of padding alone); the last
// round's K best go to val_out (may be NULL) and idx_out, padded with -infinity
// and the largest index.  scratch: 2 * topk_scratch_elems(count, K) doubles and as
// many indices.
template <typename I>
static hipError_t topk_rounds(const double *val, const I *idx, int64_t count, int K, void *scratch,
                              double *val_out, I *idx_out, hipStream_t s) {
    const int64_t sc = topk_scratch_elems(count, K);
    double *v[2] = {(double *)scratch, (double *)scratch + sc};
    I *ix[2] = {(I *)((double *)scratch + 2 * sc), (I *)((double *)scratch + 2 * sc) + sc};
    for (int side = 0;; side ^= 1) {
        const int64_t blocks = count > 0 ? cdiv(count, kChunk) : 1;
        const bool last = blocks == 1;
        hipLaunchKernelGGL(k_topk<I>, dim3((unsigned)blocks), dim3(kChunk), 0, s, val, idx, count, K,
                           last ? val_out : v[side], last ? idx_out : ix[side]);
        const hipError_t e = hipGetLastError();
        if (last || e != hipSuccess) return e;
        val = v[side];
        idx = ix[side];
        count = blocks * K;
    }
}

hipError_t launch_topk(const double *F, int64_t m, int K, void *scratch, int32_t *out,
                       hipStream_t s) {
    if (K <= 0) return hipSuccess;
    return topk_rounds<int32_t>(F, nullptr, m, K, scratch, nullptr, out, s);
}

// Round `round` of every pair of a sequence (`per` workgroups each; a pair
// whose rounds are over, or has fewer chunks, leaves them at once).  The
// signature embeddings are done with by then: their memory is the scratch.
__global__ __launch_bounds__(kChunk) void k_topk_grouped(const BatchPair *pairs, int round, int per,
                                                         int top_k) {
    __shared__ TopkShared<int32_t> sh;
    const BatchPair &q = pairs[blockIdx.x / per];
    const int64_t b = blockIdx.x % per;
    const int K = q.m < top_k ? (int)q.m : top_k;
    int64_t count = q.m;
    for (int l = 0; l < round; ++l) {
        const int64_t blocks = cdiv(count, kChunk);
        if (blocks == 1) return;
        count = blocks * K;
    }
    const int64_t blocks = cdiv(count, kChunk), sc = cdiv(q.m, kChunk) * K;
    if (b >= blocks) return;
    const int side = round & 1;
    double *v = q.Zh;
    int32_t *ix = (int32_t *)(v + 2 * sc);
    topk_chunk<int32_t>(round ? v + (side ^ 1) * sc : q.F, round ? ix + (side ^ 1) * sc : nullptr, count,
                        K, blocks == 1 ? nullptr : v + side * sc, blocks == 1 ? q.top : ix + side * sc,
                        b, sh);
}

hipError_t launch_topk_grouped(const BatchPair *pairs, const int64_t *m, int P, int top_k,
                               hipStream_t s) {
    std::vector<int64_t> count(m, m + P);
    for (int round = 0;; ++round) {
        int64_t per = 0;   // the most chunks of a pair that is not done
        for (int p = 0; p < P; ++p) {
            if (count[p] == 0) continue;
            const int64_t blocks = cdiv(count[p], kChunk);
            per = std::max(per, blocks);
            count[p] = blocks == 1 ? 0 : blocks * std::min<int64_t>(top_k, m[p]);
        }
        if (per == 0) return hipSuccess;
        hipLaunchKernelGGL(k_topk_grouped, dim3((unsigned)(per * P)), dim3(kChunk), 0, s, pairs, round,
                           (int)per, top_k);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
}

hipError_t launch_topk64(const double *val, const int64_t *idx, int64_t count, int K, void *scratch,
                         double *val_out, int64_t *idx_out, hipStream_t s) {
    return topk_rounds<int64_t>(val, idx, count, K, scratch, val_out, idx_out, s);
}

__global__ void k_edge_split(const int64_t *idx, int64_t m, int K, int32_t *a, int32_t *b) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= K) return;
    const int64_t v = idx[t];
    a[t] = (int32_t)(v / m);
    b[t] = (int32_t)(v % m);
}

hipError_t launch_edge_split(const int64_t *idx, int64_t m, int K, int32_t *a, int32_t *b,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_edge_split, dim3((unsigned)cdiv(K, 256)), dim3(256), 0, s, idx, m, K, a, b);
    return hipGetLastError();
}

} // namespace cdl
