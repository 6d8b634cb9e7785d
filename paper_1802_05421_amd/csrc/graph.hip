// Graph construction for one snapshot (Section "Climate Data": fully
// connected graph with Gaussian-kernel weights of the distance between node
// series; Background: symmetric A, no self-edges, volume V_G = sum_i D(i,i)).
//
//   pad_series   copy X into a zero-padded FP64 panel, row norms ||x_i||^2
//   gram_dist    D2_ij = ||x_i||^2 + ||x_j||^2 - 2 x_i.x_j on FP64 MFMA,
//                128 x 128 or 64 x 64 tiles covering the upper triangle
//                (nothing reads what lies below it), stored from the
//                accumulators
//   select       exact lower median of D2 over i < j: a sampled bracket
//                around the median rank, the keys inside it gathered into a
//                buffer and ranked by radix passes over their IEEE-754 bit
//                patterns (order-preserving for D2 >= 0); the same radix
//                passes over the upper triangle's keys inside the bracket when
//                the buffer does not hold them, over all of it when the
//                bracket misses the rank
//   exp_sym      per upper 64 x 64 tile: W = exp(-D2 / sigma^2) in place,
//                W_ii = 0, written with its mirror; row and column sums
//                into one partial per (tile column, node)
//   degree       deg = sum of the partials in tile order
//   graph_stats  vol = sum deg, min and max degree (fixed-order reductions)
//
// Streamed snapshots (no n x n matrix stored) use the same tiles on row
// panels: gram_dist over the panel's upper tiles (median sweeps) or all of
// its tiles, optionally with the weights formed in the epilogue; select by a
// sampled bracket gathered in one sweep over the upper panels, or by one sweep per
// radix digit;
// exp_rows for the weights, degrees and Frobenius rows of a panel.
#include "batch.h"
#include "common.h"
#include "gemm.h"
#include "kernels.h"

namespace cdl {

int64_t pad_n(int64_t n) { return ld_of(n); }
int64_t pad_k(int64_t k) { return kpad_of(k); }
int64_t pad_t(int64_t T) { return (T + 15) / 16 * 16; }

// Deterministic sum over a 64-lane wave (xor butterfly, same order everywhere).
__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Deterministic sum over a 256-thread block; result valid in every thread.
__device__ inline double block_sum256(double v, double *red) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// Whether this workgroup is the last of nb to come here (the ticket is 0
// before the first and after the last); what the others wrote before is then
// visible to it.  Every wave first waits until its own stores and atomics have
// reached the L2 (the barrier alone waits for LDS only); one thread's release
// then publishes them for the whole workgroup, since a release per wave writes
// the L2 back as often (25 against 8 us for 256 workgroups).  Every thread must
// call; `last` is a shared word.
__device__ __forceinline__ bool last_workgroup(unsigned int *ticket, unsigned int nb, int *last) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        *last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nb - 1u;
        if (*last) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            *ticket = 0u;
        }
    }
    __syncthreads();
    return *last != 0;
}

// ---------------------------------------------------------------------------

__global__ void k_fill_zero(uint4 *p, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (bytes % 16 || ((uintptr_t)p) % 16) return hipErrorInvalidValue;
    size_t n16 = bytes / 16;
    int grid = (int)(n16 / 256 + 1 < 8192 ? n16 / 256 + 1 : 8192);
    hipLaunchKernelGGL(k_fill_zero, dim3(grid), dim3(256), 0, s, (uint4 *)p, n16);
    return hipGetLastError();
}

// Small results into pinned host memory, every read in one launch: a copy
// command waits about 10 us before it starts, this kernel as long as any other.
__global__ __launch_bounds__(256) void k_read_out(ReadOut r) {
    const uint32_t *src = r.src[blockIdx.y];
    uint32_t *dst = r.dst[blockIdx.y];
    for (size_t q = (size_t)blockIdx.x * 256 + threadIdx.x; q < r.words[blockIdx.y]; q += (size_t)gridDim.x * 256)
        dst[q] = src[q];
}

hipError_t launch_read_out(const ReadOut &r, hipStream_t s) {
    size_t most = 0;
    for (int q = 0; q < r.count; ++q) most = r.words[q] > most ? r.words[q] : most;
    if (most == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((most + 1023) / 1024 < 64 ? (most + 1023) / 1024 : 64);
    hipLaunchKernelGGL(k_read_out, dim3(blocks, (unsigned)r.count), dim3(256), 0, s, r);
    return hipGetLastError();
}

// Plain device copy: one 16-byte element per lane, a grid covering the whole
// buffer (consecutive workgroups stream consecutive memory), nontemporal
// loads and stores (the data is touched once).  The reference stream for HBM
// bandwidth and for the byte counters; measured on gfx950 at 1 GiB it moves
// about 1.5x the bytes per second of a grid-stride loop over the same data.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_copy16(const u32x4 *__restrict__ src,
                                                u32x4 *__restrict__ dst, size_t n16) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n16) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

hipError_t launch_copy16(const void *src, void *dst, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (bytes % 16 || ((uintptr_t)src) % 16 || ((uintptr_t)dst) % 16) return hipErrorInvalidValue;
    const size_t n16 = bytes / 16, grid = (n16 + 255) / 256;
    if (grid > 0xffffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)grid), dim3(256), 0, s, (const u32x4 *)src,
                       (u32x4 *)dst, n16);
    return hipGetLastError();
}

// Padded row i of the series and its squared norm (one wave).
__device__ __forceinline__ void pad_row(const double *X, int64_t n, int64_t T, int64_t ldx,
                                        double *Xp, int64_t Tp, double *sqn, int *flags,
                                        int64_t i) {
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    int bad = 0;
    for (int64_t t = lane; t < Tp; t += 64) {
        double v = (i < n && t < T) ? X[i * ldx + t] : 0.0;
        if (!isfinite(v)) bad = 1;
        Xp[i * Tp + t] = v;
        s += v * v;
    }
    s = wave_sum(s);
    if (lane == 0) sqn[i] = s;
    if (flags && bad) atomicOr(flags, 1);
}

// Four rows per workgroup; ticket != nullptr: cleared for the degrees' count.
__global__ __launch_bounds__(256) void k_pad_series(const double *X, int64_t n, int64_t T, int64_t ldx,
                                                    double *Xp, int64_t Tp, double *sqn, int *flags,
                                                    int *ticket) {
    if (ticket && blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;
    pad_row(X, n, T, ldx, Xp, Tp, sqn, flags, (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6));
}

hipError_t launch_pad_series(const double *X, int64_t n, int64_t T, int64_t ldx,
                             double *Xp, int64_t rows, int64_t Tp, double *sqn,
                             int *flags, int *ticket, hipStream_t s) {
    if (rows % 4) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pad_series, dim3((unsigned)(rows / 4)), dim3(256), 0, s, X, n, T, ldx, Xp,
                       Tp, sqn, flags, ticket);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Squared distances from the Gram matrix of the series (FP64 MFMA).

// Tile shapes (the same bits from each).  0: 128 x 128 by eight waves, two
// workgroups on a CU; the cover's 256 x 128 tiles (whose order shares operand
// panels in an XCD's L2) are each computed as two such halves.  1: 64 x 64 by
// four waves, three on a CU, for sizes that 128 x 128 tiles cannot spread over
// the CUs.  2: the same with 64-bit addresses, for very long series.  What a tile costs beside its MFMAs (2 n^2 T / 2 flop in all) is
// the first loads and the epilogue: distances, median bracket, stores; other
// workgroups' MFMAs run beside them.
template <int SHAPE> struct GramCfg;
template <> struct GramCfg<0> {
    using Core = Dma64Core<128, 128, 2, 4, 2>;
    static constexpr int WAVES = 4;   // waves per SIMD that the registers leave room for
};
template <> struct GramCfg<1> {
    using Core = Dma64Core<64, 64, 2, 2, 3>;
    static constexpr int WAVES = 3;
};
template <> struct GramCfg<2> {
    using Core = Dma64Core<64, 64, 2, 2, 3, true>;
    static constexpr int WAVES = 3;
};
// Padded series lengths from which shape 2 takes over: 128 rows of 2^22 values
// are 2^32 bytes, the reach of the other shapes' offsets.
constexpr int64_t kGramFar = (int64_t)1 << 22;
// What a launch covers: the upper triangle of the whole matrix, the upper
// triangle's part of a row panel, or a whole row panel: its upper part, whose
// tiles in the panel's own square are also stored mirrored (the same bits; half
// of a sweep's Gram where one panel holds every row, a fifth at n = 20000 with
// panels of 8192), and the columns before that square.
enum GramCover { kGramUpper, kGramPanelUpper, kGramPanelFull };

// Workgroups of shape `shape` on rows [row0, row0 + rows) (multiples of 256).
static int64_t gram_wgs(int shape, GramCover cover, int64_t ld, int64_t row0, int64_t rows) {
    if (shape == 0) return 2 * gram_panel_tiles(ld, row0, rows, cover == kGramPanelFull);
    const int64_t nt = ld / 64;
    if (cover == kGramUpper) return nt * (nt + 1) / 2;
    return rows / 64 * (cover == kGramPanelFull ? nt : (ld - row0) / 64);   // (some without a tile)
}

// The busiest CU's work in 64 x 64 tiles: the small tiles' rate is 0.8 of the
// large ones' (twice the first loads and operand traffic per flop).
static int gram_shape(GramCover cover, int64_t ld, int64_t Tp, int64_t row0, int64_t rows) {
    if (Tp >= kGramFar) return 2;
    const double t0 = 4.0 * (double)cdiv(gram_wgs(0, cover, ld, row0, rows), 256);
    const double t1 = (double)cdiv(gram_wgs(1, cover, ld, row0, rows), 256) / 0.8;
    return t1 < t0 ? 1 : 0;
}

// First row and column of workgroup `id` (after the XCD remap); false: no tile.
template <int SHAPE>
__device__ inline bool gram_place(int cover, int id, int64_t ld, int64_t row0, int64_t rows,
                                  int64_t &m0, int64_t &n0) {
    int I, J;
    if (SHAPE == 0) {
        const int tile = id >> 1, half = id & 1, I0 = (int)(row0 / 256), pb = (int)(rows / 256);
        const int ncol = (int)(ld / 128), upper = pb * ncol - 2 * (I0 * pb + pb * (pb - 1) / 2);
        if (tile < upper) {
            upper_band_tile<4>(tile, I0, pb, ncol, I, J);
        } else {
            rect_tile<4>(tile - upper, pb, 2 * I0, I, J);
            I += I0;
        }
        m0 = (int64_t)I * 256 + 128 * half;
        n0 = (int64_t)J * 128;
        // (the lower halves of a panel's 256-row diagonal tiles: their mirror)
        return cover != kGramPanelFull || tile >= upper || n0 >= m0;
    }
    if (cover == kGramUpper) {
        sym_tile<8>(id, (int)(ld / 64), I, J);
        m0 = (int64_t)I * 64;
        n0 = (int64_t)J * 64;
        return true;
    }
    const int pb = (int)(rows / 64), I0 = (int)(row0 / 64), right = (int)(ld / 64) - I0;
    if (id < pb * right) {
        rect_tile<8>(id, pb, right, I, J);
        J += I0;
    } else {
        rect_tile<8>(id - pb * right, pb, I0, I, J);
    }
    I += I0;
    m0 = (int64_t)I * 64;
    n0 = (int64_t)J * 64;
    return id >= pb * right || I <= J;
}

// One tile.  Row i is stored at D2 + (i - row0) ld, so a row panel needs a
// buffer of its own rows only.
// st != nullptr: also fold the smallest and largest upper-triangle key
// (i < j) into st->kmin / st->kmax (the median selection starts below their
// common bit prefix); with brbuf as well, the bracket pass of the selection
// on the tile's upper-triangle keys: count those below st->lo into st->below
// and append those in [lo, hi] to brbuf (capacity brcap) through an LDS
// stage in the GEMM's staging memory, one segment per wave (a wave with more
// of them than its segment holds counts them, marks the buffer unusable and the
// selection passes over the matrix: exact either way).  Each lane counts
// its own keys below and up to the bracket's end, one scan over the wave gives
// its place, and a second walk over its registers appends them (a ballot and a
// popcount per element before: the epilogue took half of a launch at T = 120).
// NaN distances (non-finite series) are stored and left out of the selection.
// kExp: store the weights exp(-D2 / sigma^2) instead (zero on the diagonal and
// outside n; sigma = wstats[1]), the expression of the separate exponential
// kernels, so the values are the same bits.
// kPanel: a whole row panel (kGramPanelFull).
template <int SHAPE, bool kExp, bool kPanel>
__device__ __forceinline__ void gram_tile(const double *Xp, int64_t Tp, const double *sqn,
                                          int64_t n, int64_t ld, double *D2, int64_t row0,
                                          int64_t rows, int cover, int id, SelectState *st,
                                          const double *wstats, double *smem,
                                          unsigned long long *brbuf = nullptr,
                                          int64_t brcap = 0) {
    using Core = typename GramCfg<SHAPE>::Core;
    constexpr int R = MfmaF64::R;
    int64_t m0, n0;
    if (!gram_place<SHAPE>(cover, id, ld, row0, rows, m0, n0)) return;
    // the bracket and the extremes so far, read before the MFMAs hide it (an
    // extreme that has moved since costs an atomic more, nothing else)
    const unsigned long long kInf = 0x7ff0000000000000ull;
    double lo = 0.0, hi = -1.0;   // no bracket: nothing below, nothing inside
    unsigned long long kmin0 = 0ull, kmax0 = 0ull;
    if (!kExp && st) {
        kmin0 = st->kmin;
        kmax0 = st->kmax;
        if (brbuf) {
            lo = __longlong_as_double((long long)st->lo);
            hi = __longlong_as_double((long long)(st->hi > kInf ? kInf : st->hi));
        }
    }
    Core g;
    g.run(Xp, Tp, Xp, Tp, m0, n0, Tp, smem);
    double *const out = D2 - row0 * ld;
    // the squared norms of this lane's rows and columns, loaded once (the
    // stores below may alias sqn as far as the compiler knows)
    double sa[Core::WTM][R], sb[Core::WTN];
#pragma unroll
    for (int a = 0; a < Core::WTM; ++a)
#pragma unroll
        for (int rr = 0; rr < R; ++rr) sa[a][rr] = sqn[m0 + Core::row_of(a, rr)];
#pragma unroll
    for (int b = 0; b < Core::WTN; ++b) sb[b] = sqn[n0 + Core::col_of(b)];
    double s2 = 0.0;
    if (kExp) {
        const double sigma = wstats[1];
        s2 = sigma * sigma;
    }
    // distances, stored as 16 lanes' 16 consecutive columns of one row; the
    // accumulators keep the upper-triangle keys (NaN: not one)
    const int ni = (int)n, mi = (int)m0, nj = (int)n0;   // n < 2^20
#pragma unroll
    for (int a = 0; a < Core::WTM; ++a) {
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
            const int i = mi + Core::row_of(a, rr);
            double *const row = out + (int64_t)i * ld + n0;
#pragma unroll
            for (int b = 0; b < Core::WTN; ++b) {
                const int c = Core::col_of(b), j = nj + c;
                double d = sa[a][rr] + sb[b] - 2.0 * g.acc[a][b][rr];
                d = d < 0.0 ? 0.0 : d;
                const bool pair = i < ni && j < ni && i != j;
                d = pair ? d : 0.0;
                if (kExp) d = pair ? exp(-d / s2) : 0.0;
                g.acc[a][b][rr] = kPanel || (pair && i < j) ? d : NAN;
                row[c] = d;
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // bounds the addresses and masks held at once
    }
    if (kPanel) {
        // (four lanes make 32 consecutive bytes of the mirror, the four stores of a
        // lane a line of it)
        if (n0 > m0 && n0 < row0 + rows)
#pragma unroll
            for (int b = 0; b < Core::WTN; ++b) {
                double *const row = out + (n0 + Core::col_of(b)) * ld + m0;
#pragma unroll
                for (int a = 0; a < Core::WTM; ++a)
#pragma unroll
                    for (int rr = 0; rr < R; ++rr) row[Core::row_of(a, rr)] = g.acc[a][b][rr];
                __builtin_amdgcn_sched_barrier(0);
            }
        return;
    }
    if (kExp || !st) return;

    __shared__ double wmin[Core::NW], wmax[Core::NW];
    __shared__ unsigned int wbel[Core::NW], wcnt[Core::NW];
    __shared__ unsigned long long sbase;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    double kmin = INFINITY, kmax = -1.0;
    unsigned int below = 0, upto = 0;   // this lane's keys < lo and <= hi
#pragma unroll
    for (int a = 0; a < Core::WTM; ++a)
#pragma unroll
        for (int b = 0; b < Core::WTN; ++b)
#pragma unroll
            for (int rr = 0; rr < R; ++rr) {
                const double d = g.acc[a][b][rr];
                kmin = fmin(kmin, d);
                kmax = fmax(kmax, d);
                below += d < lo ? 1u : 0u;
                upto += d <= hi ? 1u : 0u;
            }
    const unsigned int mine = brbuf ? upto - below : 0u;
    unsigned int pos = mine, bw = below;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int y = __shfl_up(pos, o);
        pos += lane >= o ? y : 0u;
    }
    const unsigned int count = __shfl(pos, 63);   // the wave's keys inside
    pos -= mine;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        kmin = fmin(kmin, __shfl_xor(kmin, o));
        kmax = fmax(kmax, __shfl_xor(kmax, o));
        bw += __shfl_xor(bw, o);
    }
    if (lane == 0) {
        wmin[wid] = kmin;
        wmax[wid] = kmax;
        wbel[wid] = bw;
        wcnt[wid] = count;
    }
    __syncthreads();
    unsigned long long tbase = 0ull;
    // the GEMM's LDS is free: one segment of it per wave
    constexpr unsigned int kSeg = (unsigned int)(Core::SMEM / 8 / Core::NW);
    if (threadIdx.x == 0) {
        // Every tile updates the same few words, and such an atomic takes about
        // 8 ns whoever asks: so one per tile for the buffer's length, the count
        // below spread over 64 lines, and the extremes only where they move.
        unsigned long long bl = 0ull, cnt = 0ull;
        bool over = false;
#pragma unroll
        for (int w = 0; w < Core::NW; ++w) {
            kmin = fmin(kmin, wmin[w]);
            kmax = fmax(kmax, wmax[w]);
            bl += wbel[w];
            cnt += wcnt[w];
            over = over || wcnt[w] > kSeg;
        }
        if (kmax >= 0.0) {   // the tile holds a key
            const unsigned long long k0 = (unsigned long long)__double_as_longlong(kmin);
            const unsigned long long k1 = (unsigned long long)__double_as_longlong(kmax);
            if (k0 < kmin0) atomicMin(&st->kmin, k0);
            if (k1 > kmax0) atomicMax(&st->kmax, k1);
        }
        if (cnt) tbase = atomicAdd(&st->nbuf, cnt);
        if (over) atomicOr(&st->over, 1u);
        if (bl) atomicAdd(&st->part[(blockIdx.x % kBelowParts) * kBelowPitch], bl);
    }
    if (!brbuf) return;
    if (count <= kSeg) {   // uniform over the wave
        unsigned long long *const seg = (unsigned long long *)smem + wid * kSeg;
        // (opaque copies: the tests are made again rather than kept as masks)
        double lo2 = lo, hi2 = hi;
        asm volatile("" : "+v"(lo2), "+v"(hi2));
#pragma unroll
        for (int a = 0; a < Core::WTM; ++a) {
#pragma unroll
            for (int b = 0; b < Core::WTN; ++b)
#pragma unroll
                for (int rr = 0; rr < R; ++rr) {
                    const double d = g.acc[a][b][rr];
                    if (d >= lo2 && d <= hi2)
                        seg[pos++] = (unsigned long long)__double_as_longlong(d);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (threadIdx.x == 0) sbase = tbase;   // (asked for before the segment was filled)
    __syncthreads();
    unsigned long long base = sbase;
    for (int w = 0; w < wid; ++w) base += wcnt[w];
    // (a full segment has marked the buffer unusable: its wave has nothing to copy)
    if (count <= kSeg) {
        const unsigned long long *const seg = (const unsigned long long *)smem + wid * kSeg;
        for (unsigned int q = lane; q < count; q += 64)
            if (base + q < (unsigned long long)brcap) brbuf[base + q] = seg[q];
    }
}

template <int SHAPE, bool kExp, bool kPanel>
__global__ __launch_bounds__(GramCfg<SHAPE>::Core::NT, GramCfg<SHAPE>::WAVES) void k_gram_dist(
    const double *Xp, int64_t Tp, const double *sqn, int64_t n, int64_t ld, double *D2,
    int64_t row0, int64_t rows, int cover, SelectState *st, const double *wstats,
    unsigned long long *brbuf, int64_t brcap) {
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    gram_tile<SHAPE, kExp, kPanel>(Xp, Tp, sqn, n, ld, D2, row0, rows, cover, xcd_remap(blockIdx.x, gridDim.x),
                           st, wstats, (double *)smem_raw, brbuf, brcap);
}

template <int SHAPE, bool kExp, bool kPanel>
static hipError_t gram_launch(const double *Xp, int64_t Tp, const double *sqn, int64_t n, int64_t ld,
                              double *D2, int64_t row0, int64_t rows, GramCover cover,
                              SelectState *st, const double *wstats, unsigned long long *brbuf,
                              int64_t brcap, hipStream_t s) {
    using Core = typename GramCfg<SHAPE>::Core;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void *)k_gram_dist<SHAPE, kExp, kPanel>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)Core::SMEM);
        if (e != hipSuccess) return e;
        attr = true;
    }
    const int64_t total = gram_wgs(SHAPE, cover, ld, row0, rows);
    if (total <= 0 || total > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gram_dist<SHAPE, kExp, kPanel>), dim3((unsigned)total), dim3(Core::NT), Core::SMEM,
                       s, Xp, Tp, sqn, n, ld, D2, row0, rows, (int)cover, st, wstats, brbuf, brcap);
    return hipGetLastError();
}

template <bool kExp, bool kPanel>
static hipError_t gram_any(const double *Xp, int64_t Tp, const double *sqn, int64_t n, int64_t ld, double *D2,
                           int64_t row0, int64_t rows, GramCover cover, SelectState *st,
                           const double *wstats, unsigned long long *brbuf, int64_t brcap, hipStream_t s) {
    switch (gram_shape(cover, ld, Tp, row0, rows)) {
    case 0: return gram_launch<0, kExp, kPanel>(Xp, Tp, sqn, n, ld, D2, row0, rows, cover, st, wstats, brbuf, brcap, s);
    case 1: return gram_launch<1, kExp, kPanel>(Xp, Tp, sqn, n, ld, D2, row0, rows, cover, st, wstats, brbuf, brcap, s);
    default: return gram_launch<2, kExp, kPanel>(Xp, Tp, sqn, n, ld, D2, row0, rows, cover, st, wstats, brbuf, brcap, s);
    }
}

hipError_t launch_gram_dist(const double *Xp, int64_t Tp, const double *sqn, int64_t n,
                            int64_t ld, double *D2, SelectState *st, unsigned long long *brbuf,
                            int64_t brcap, hipStream_t s) {
    if (brbuf && !st) return hipErrorInvalidValue;
    return gram_any<false, false>(Xp, Tp, sqn, n, ld, D2, 0, ld, kGramUpper, st, nullptr, brbuf, brcap, s);
}

int64_t gram_panel_tiles(int64_t ld, int64_t row0, int64_t rows, bool full) {
    const int64_t ncol = ld / 128, I0 = row0 / 256, pb = rows / 256;
    return pb * ncol - 2 * (I0 * pb + pb * (pb - 1) / 2) + (full ? 2 * I0 * pb : 0);
}

hipError_t launch_gram_panel(const double *Xp, int64_t Tp, const double *sqn, int64_t n,
                             int64_t ld, int64_t row0, int64_t rows, bool full, double *D2p,
                             const double *wstats, hipStream_t s) {
    if (row0 % 256 || rows % 256 || rows <= 0 || row0 + rows > ld) return hipErrorInvalidValue;
    if (wstats && !full) return hipErrorInvalidValue;
    const GramCover cover = full ? kGramPanelFull : kGramPanelUpper;
    if (wstats) return gram_any<true, true>(Xp, Tp, sqn, n, ld, D2p, row0, rows, cover, nullptr, wstats, nullptr, 0, s);
    if (full) return gram_any<false, true>(Xp, Tp, sqn, n, ld, D2p, row0, rows, cover, nullptr, nullptr, nullptr, 0, s);
    return gram_any<false, false>(Xp, Tp, sqn, n, ld, D2p, row0, rows, cover, nullptr, nullptr, nullptr, 0, s);
}

// ---------------------------------------------------------------------------
// Exact selection of the element of rank floor((N-1)/2), N = n(n-1)/2, among
// D2_ij (i < j).  D2 >= 0, so its IEEE bit pattern orders like its value.
// First a bracket: the sample quantiles three standard deviations on each side
// of the target, of pairs whose distances are taken from the series before the
// Gram, widened by what the rounding of two orders of summation can differ; the
// keys below lo are counted and those in [lo, hi] counted and appended to a
// buffer, by the Gram's epilogue for stored snapshots, by one sweep over the
// recomputed upper panels for streamed ones.  If the target rank falls inside
// the bracket the radix passes below run over the buffer, or, where many keys
// crowd there and it does not hold them, over the matrix's keys inside the
// bracket; else over the whole matrix (the result is exact either way).  Inside a
// bracket a pass takes its digit from key - lo, of which hi - lo leaves few bits:
// distances that differ by rounding alone (patterns that repeat) are resolved by
// one digit, where digits of the keys themselves took a pass over the matrix for
// every 12 of the 40 leading bits that such keys share; and where a pass finds that
// all its keys share more bits than its digit, the next digit starts behind them
// (such a crowd beside zeros: 0.36 ms a graph at n = 4096, 11.9 without).  A digit
// has 12 bits; as soon as the selected bin holds at most kSelFew keys, one pass
// collects them and counting ranks among them gives the answer.  The last workgroup
// of a pass picks the digit, so a pass is one launch; every pass reads the state's
// mode, so the fixed launch sequence turns into no-ops once the answer is
// known.  Launch latency and single-workgroup steps bound all of this: six
// launches and 55 us of a graph at n = 4096 (100 at n = 16384), where 21
// launches with a sort of the sample, a sort of the candidates and a pick of
// their own took 177 (192).

constexpr int kSelFew = 512;      // candidates ranked by the last pass's last workgroup
static_assert(kSelFew <= kSelCap, "candidates must fit the state");
constexpr int kSelSmall = 512;    // nodes (131k keys) up to which one workgroup does it all

__device__ __forceinline__ void select_reset_body(SelectState *st) {
    for (int b = threadIdx.x; b < 4096; b += blockDim.x) st->hist[b] = 0;
    if (threadIdx.x == 0) {
        st->kmin = ~0ull;
        st->kmax = 0ull;
        st->count = 0;
        st->mode = 0;
        st->src = 0;
        st->below = 0;
        st->nbuf = 0;
        st->ticket = 0;
        st->over = 0;
        st->kand = ~0ull;
        st->kor = 0ull;
    }
    for (int q = threadIdx.x; q < kBelowParts; q += blockDim.x) st->part[q * kBelowPitch] = 0;
}

__global__ void k_select_reset(SelectState *st) { select_reset_body(st); }

// Before the ranks of a sample: the bracket's ends are found as minima and maxima.
__device__ __forceinline__ void select_bracket_reset(SelectState *st) {
    if (threadIdx.x == 0) {
        st->lo = ~0ull;
        st->hi = 0ull;
    }
}

constexpr int kSelSample = 4096;  // (and kStreamSample: multiples of kRankTile)
constexpr int kSelMargin = 96;    // 3 sqrt(kSelSample / 4): misses in ~0.3% of calls

int64_t select_buffer_keys(int64_t n) {
    const int64_t N = n * (n - 1) / 2;
    const int64_t cap = N / 8 + 65536;
    return cap < ((int64_t)1 << 27) ? cap : ((int64_t)1 << 27);
}

__device__ inline unsigned long long sel_mix(unsigned long long z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Sample pair u of the bracket: a pseudo-random pair i != j.
__device__ inline void sel_pair(unsigned long long u, int64_t n, int64_t &a, int64_t &b) {
    const unsigned long long h = sel_mix(0x5851f42d4c957f2dull + u);
    const int64_t i = (int64_t)((h & 0xffffffffull) % (unsigned long long)n);
    int64_t j = (int64_t)((h >> 32) % (unsigned long long)(n - 1));
    if (j >= i) ++j;   // j != i
    a = i < j ? i : j;
    b = i < j ? j : i;
}

// Keys of the sample pairs from the padded series, before the Gram: one wave
// per pair, D2 = sq_a + sq_b - 2 x_a.x_b with the dot product summed over the
// lanes (another order than the Gram's: an estimate of the quantile, which is
// all the bracket needs; the counts against it are exact).  Four pairs a wave
// (sixteen where the snapshots of a group fill the chip): each costs a round trip
// to memory, so they are spread over the whole chip.
__device__ __forceinline__ void select_sample_keys_body(const double *Xp, int64_t Tp,
                                                        const double *sqn, int64_t n, int samples,
                                                        unsigned long long *keys, int wave,
                                                        int nwave) {
    const int lane = threadIdx.x & 63;
    for (int u = wave; u < samples; u += nwave) {
        int64_t a, b;
        sel_pair((unsigned long long)u, n, a, b);
        const double *xa = Xp + a * Tp, *xb = Xp + b * Tp;
        double dot = 0.0;
        for (int64_t q = lane; q < Tp; q += 64) dot += xa[q] * xb[q];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) dot += __shfl_xor(dot, o);
        if (lane == 0) {
            double d = sqn[a] + sqn[b] - 2.0 * dot;
            d = d < 0.0 ? 0.0 : d;
            keys[u] = (unsigned long long)__double_as_longlong(d);
        }
    }
}

// Sample keys; the first workgroup also resets the selection state.
__global__ __launch_bounds__(256) void k_select_sample_keys(const double *Xp, int64_t Tp,
                                                            const double *sqn, int64_t n, int samples,
                                                            unsigned long long *keys,
                                                            SelectState *st) {
    if (blockIdx.x == 0) {
        select_reset_body(st);
        select_bracket_reset(st);
    }
    select_sample_keys_body(Xp, Tp, sqn, n, samples, keys, blockIdx.x * 4 + (threadIdx.x >> 6),
                            gridDim.x * 4);
}

// The bracket [lo, hi]: the sample keys of ranks q -/+ margin around the
// target quantile's rank q, moved outwards by the difference that the rounding of
// the sample's and of the Gram's order of summation can make (without that, a
// crowd of distances that are equal but for rounding could lie beside its own
// sample's bracket).  Workgroup b ranks keys 64 b .. 64 b + 63 against
// the whole sample, 4096 keys of it at a time in LDS, a sixteenth of those per
// wave (every lane reads the same two keys): a key's rank is the number of
// smaller keys (equal keys hold a run of ranks, and the outermost end counts).
constexpr int kRankTile = 4096;

// Bound of that difference for pair u: each order rounds a sum of Tp products at
// most Tp + 16 times, |x_a| |x_b| <= (sq_a + sq_b) / 2.
__device__ inline double select_slack(int64_t u, int64_t n, const double *sqn, int64_t Tp) {
    int64_t a, b;
    sel_pair((unsigned long long)u, n, a, b);
    return (double)(Tp + 16) * 0x1p-52 * (sqn[a] + sqn[b]);
}

__device__ __forceinline__ void select_rank_body(const unsigned long long *keys, int samples,
                                                 int margin, int64_t n, const double *sqn, int64_t Tp,
                                                 SelectState *st, int b) {
    struct alignas(16) Two { unsigned long long x, y; };
    __shared__ Two tile[kRankTile / 2];
    __shared__ unsigned int less[16][64], upto[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long mine = keys[64 * b + lane];
    unsigned int lt = 0, le = 0;
    for (int j0 = 0; j0 < samples; j0 += kRankTile) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRankTile / 2048; ++q)
            tile[threadIdx.x + 1024 * q] = ((const Two *)(keys + j0))[threadIdx.x + 1024 * q];
        __syncthreads();
        const Two *part = tile + w * (kRankTile / 32);
#pragma unroll 8
        for (int j = 0; j < kRankTile / 32; ++j) {
            const Two k = part[j];
            lt += k.x < mine ? 1u : 0u;
            le += k.x <= mine ? 1u : 0u;
            lt += k.y < mine ? 1u : 0u;
            le += k.y <= mine ? 1u : 0u;
        }
    }
    less[w][lane] = lt;
    upto[w][lane] = le;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    lt = le = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        lt += less[q][lane];
        le += upto[q][lane];
    }
    const unsigned long long N = (unsigned long long)n * (unsigned long long)(n - 1) / 2ull;
    const double rho = (double)((N - 1ull) / 2ull) / (double)N;
    const int q = (int)(rho * samples), rlo = q - margin, rhi = q + margin;
    // (a NaN among the ends stays what it is)
    const double d = __longlong_as_double((long long)mine);
    if (rlo > 0) {
        if ((int)lt <= rlo && rlo < (int)le) {
            const double x = d - select_slack(64 * b + lane, n, sqn, Tp);
            atomicMin(&st->lo, x > 0.0 ? (unsigned long long)__double_as_longlong(x) : x <= 0.0 ? 0ull : mine);
        }
    } else if (b == 0 && lane == 0) {
        atomicMin(&st->lo, 0ull);
    }
    if (rhi < samples - 1) {
        if ((int)lt <= rhi && rhi < (int)le) {
            const double x = d + select_slack(64 * b + lane, n, sqn, Tp);
            atomicMax(&st->hi, x >= d ? (unsigned long long)__double_as_longlong(x) : mine);
        }
    } else if (b == 0 && lane == 0) {
        atomicMax(&st->hi, ~0ull);
    }
}

__global__ __launch_bounds__(1024) void k_select_rank(const unsigned long long *keys, int samples,
                                                      int margin, int64_t n, const double *sqn,
                                                      int64_t Tp, SelectState *st) {
    select_rank_body(keys, samples, margin, n, sqn, Tp, st, blockIdx.x);
}

// The bracket pass for very many keys (streamed panels: billions of keys,
// tens of thousands inside the bracket per workgroup): the workgroup's rows
// go in rounds of 2048 keys with a barrier after each, and whenever the LDS
// stage holds 2048 or more keys it is copied out behind one global atomic,
// so the global counter sees one atomic per ~2048 keys instead of one each.
__global__ __launch_bounds__(256) void k_select_bracket_flush(const double *D2, int64_t ld,
                                                              int64_t n, int64_t row0,
                                                              int64_t row1, SelectState *st,
                                                              unsigned long long *buf,
                                                              int64_t cap) {
    constexpr unsigned int kStage = 4096, kRound = 8 * 256;
    __shared__ unsigned long long sb[kStage];
    __shared__ unsigned int scnt;
    __shared__ unsigned long long sbase, spart[4];
    if (st->mode == 2) return;
    const unsigned long long lo = st->lo, hi = st->hi;
    const int t = threadIdx.x;
    if (t == 0) scnt = 0;
    __syncthreads();
    unsigned long long below = 0;
    auto flush = [&]() {   // every thread, after a barrier
        const unsigned int c = scnt;
        if (t == 0 && c > 0) sbase = atomicAdd(&st->nbuf, (unsigned long long)c);
        __syncthreads();
        const unsigned long long base = sbase;
        for (unsigned int q = t; q < c; q += 256)
            if (base + q < (unsigned long long)cap) buf[base + q] = sb[q];
        __syncthreads();
        if (t == 0) scnt = 0;
        __syncthreads();
    };
    for (int64_t i = row0 + blockIdx.x; i < row1; i += gridDim.x) {
        const unsigned long long *row = (const unsigned long long *)(D2 + (i - row0) * ld);
        for (int64_t jb = i + 1; jb < n; jb += kRound) {   // the same trip count in every thread
            unsigned long long key[8];   // eight independent loads in flight
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t j = jb + t + 256 * u;
                key[u] = j < n ? row[j] : ~0ull;   // ~0: above every bracket
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (key[u] < lo) {
                    ++below;
                } else if (key[u] <= hi && key[u] != ~0ull) {
                    const unsigned int q = atomicAdd(&scnt, 1u);   // < kStage: at most kRound per round
                    sb[q] = key[u];
                }
            }
            __syncthreads();
            const unsigned int c = scnt;
            __syncthreads();   // read by every thread before the next round appends
            if (c >= kStage - kRound) flush();
        }
    }
    __syncthreads();
    flush();
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) below += __shfl_xor(below, o);
    if ((t & 63) == 0) spart[t >> 6] = below;
    __syncthreads();
    if (t == 0) {
        const unsigned long long b = spart[0] + spart[1] + spart[2] + spart[3];
        if (b) atomicAdd(&st->below, b);
    }
}

// The part of the state that a pass works from.  It selects among x = key - base
// of the keys with x <= span.
struct SelView {
    unsigned long long prefix, rank, base, span;
    int bits, mode, src;
};
__device__ inline SelView select_load(const SelectState *st) {
    const int src = st->src;
    const unsigned long long lo = st->lo, hi = st->hi;
    return SelView{st->prefix, st->rank, src ? lo : 0ull, src == 2 ? hi - lo : ~0ull, st->bits, st->mode, src};
}

// Move the radix passes into the bracket when the target lies there: to the
// buffer, or to the matrix's keys inside when the buffer does not hold them all.
__device__ inline void select_bracket_view(const SelectState *st, int64_t cap, SelView &v) {
    if (v.mode == 2) return;
    unsigned long long below = st->below;
    const unsigned long long nb = st->nbuf;
#pragma unroll 16
    for (int q = 0; q < kBelowParts; ++q) below += st->part[q * kBelowPitch];
    if (v.rank < below || v.rank >= below + nb) return;   // stay on the whole matrix
    const unsigned long long x = st->hi - st->lo;
    v.src = nb > (unsigned long long)cap || st->over ? 2 : 1;
    v.rank -= below;
    v.base = st->lo;
    v.span = v.src == 2 ? x : ~0ull;
    v.prefix = 0ull;
    if (x == 0ull) {   // every bracket key equals lo
        v.bits = 64;
        v.mode = 2;
        return;
    }
    v.bits = __clzll((long long)x);
    v.mode = v.src == 1 && nb <= (unsigned long long)kSelFew ? 1 : 0;
}

// The start of a stored selection: target rank and common prefix of the keys,
// then the bracket when one was gathered.  Every workgroup of the first pass
// makes it from the state while others of its launch may be passing already, so
// it reads nothing that a pass writes.
__device__ inline SelView select_start(const SelectState *st, int64_t n, int64_t cap, bool gathered) {
    SelView v;
    const unsigned long long N = (unsigned long long)n * (unsigned long long)(n - 1) / 2ull;
    v.rank = (N - 1ull) / 2ull;
    v.src = 0;
    v.base = 0ull;
    v.span = ~0ull;
    const unsigned long long x = st->kmin ^ st->kmax;
    if (x == 0ull) {   // every pair distance is the same value
        v.prefix = st->kmin;
        v.bits = 64;
        v.mode = 2;
        return v;
    }
    const int L = __clzll((long long)x);
    v.bits = L;
    v.prefix = L == 0 ? 0ull : (st->kmin & ~((1ull << (64 - L)) - 1ull));
    v.mode = 0;
    if (gathered) select_bracket_view(st, cap, v);
    return v;
}

__device__ inline void select_done(SelectState *st, double *stats, unsigned long long key) {
    st->mode = 2;
    stats[1] = sqrt(__longlong_as_double((long long)key));
}

__global__ void k_select_check(SelectState *st, int64_t cap, double *stats) {
    if (threadIdx.x != 0) return;
    SelView v = select_load(st);
    const int before = v.mode;
    select_bracket_view(st, cap, v);
    st->prefix = v.prefix;
    st->rank = v.rank;
    st->bits = v.bits;
    st->mode = v.mode;
    st->src = v.src;
    st->count = 0;
    if (v.mode == 2 && before != 2) select_done(st, stats, v.base + v.prefix);
}

__device__ inline void sel_digit(int bits, int &shift, int &width, unsigned long long &hi_mask) {
    width = 64 - bits < 12 ? 64 - bits : 12;
    shift = 64 - bits - width;
    hi_mask = bits == 0 ? 0ull : ~((1ull << (64 - bits)) - 1ull);
}

// Keys of rows [row0, row1): row i at D2 + (i - row0) ld (a row panel, or
// the whole matrix with row0 = 0, row1 = n), or of the bracket buffer.
// Workgroup b of nb adds its share to the digit's histogram (mode 0) or to the
// candidates (mode 1); NT threads.
template <int NT>
__device__ __forceinline__ void select_pass_body(const double *D2, int64_t ld, int64_t n,
                                                 int64_t row0, int64_t row1, SelectState *st,
                                                 const SelView &v, const unsigned long long *buf,
                                                 int64_t b, int64_t nb, unsigned int *h) {
    constexpr int nt = NT;
    int shift, width;
    unsigned long long hi_mask;
    sel_digit(v.bits, shift, width, hi_mask);
    const int mode = v.mode;
    const unsigned long long prefix = v.prefix;
    if (mode == 0) {
        for (int q = threadIdx.x; q < 4096; q += nt) h[q] = 0;
        __syncthreads();
    }
    const unsigned long long dmask = (1ull << width) - 1ull;
    unsigned long long kand = ~0ull, kor = 0ull;
    auto take = [&](unsigned long long key) {
        const unsigned long long x = key - v.base;
        if (x > v.span || (x & hi_mask) != prefix) return;
        if (mode == 0) {
            atomicAdd(&h[(x >> shift) & dmask], 1u);
            kand &= x;
            kor |= x;
        } else {
            const unsigned int q = atomicAdd(&st->count, 1u);
            if (q < kSelCap) st->cand[q] = x;
        }
    };
    // eight independent loads in flight per thread
    if (v.src == 1) {
        const int64_t nk = (int64_t)st->nbuf, stride = nb * nt;
        for (int64_t q0 = b * nt + threadIdx.x; q0 < nk; q0 += 8 * stride) {
            unsigned long long key[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) key[u] = q0 + u * stride < nk ? buf[q0 + u * stride] : 0ull;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q0 + u * stride < nk) take(key[u]);
        }
    } else {
        for (int64_t i = row0 + b; i < row1; i += nb) {
            const unsigned long long *row = (const unsigned long long *)(D2 + (i - row0) * ld);
            for (int64_t j0 = i + 1 + threadIdx.x; j0 < n; j0 += 8 * nt) {
                unsigned long long key[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) key[u] = j0 + nt * u < n ? row[j0 + nt * u] : 0ull;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (j0 + nt * u < n) take(key[u]);
            }
        }
    }
    if (mode == 0) {
        __syncthreads();
        for (int q = threadIdx.x; q < 4096; q += nt)
            if (h[q]) atomicAdd(&st->hist[q], (unsigned long long)h[q]);
        __syncthreads();
        // AND and OR over the workgroup (the histogram's LDS is free)
        unsigned long long *const red = (unsigned long long *)h;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            kand &= __shfl_xor(kand, o);
            kor |= __shfl_xor(kor, o);
        }
        if ((threadIdx.x & 63) == 0) {
            red[threadIdx.x >> 6] = kand;
            red[16 + (threadIdx.x >> 6)] = kor;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < nt / 64; ++w) {
                kand &= red[w];
                kor |= red[16 + w];
            }
            if (kor || kand != ~0ull) {   // a key matched
                atomicAnd(&st->kand, kand);
                atomicOr(&st->kor, kor);
            }
        }
    }
}

struct PickShared {
    unsigned long long part[16], keys[kSelFew];
};

// Pick the digit from the histogram, or the answer from the candidates, and
// write the state for the next pass.  One workgroup of NT threads.
template <int NT>
__device__ __forceinline__ void select_pick_body(SelectState *st, const SelView &v, double *stats,
                                                 PickShared &sh) {
    constexpr int nt = NT;
    const int t = threadIdx.x;
    if (v.mode == 2) return;
    if (v.mode == 1) {
        // the candidate with `rank` smaller ones (equal candidates hold a run
        // of ranks; each may write the same answer)
        const int cnt = (int)(st->count < kSelFew ? st->count : kSelFew);
        for (int q = t; q < cnt; q += nt) sh.keys[q] = st->cand[q];
        __syncthreads();
        for (int q = t; q < cnt; q += nt) {
            const unsigned long long mine = sh.keys[q];
            unsigned int lt = 0, le = 0;
            for (int j = 0; j < cnt; ++j) {
                lt += sh.keys[j] < mine ? 1u : 0u;
                le += sh.keys[j] <= mine ? 1u : 0u;
            }
            if (lt <= v.rank && v.rank < le) {
                st->prefix = mine;
                st->bits = 64;
                select_done(st, stats, v.base + mine);
            }
        }
        return;
    }
    // (many pairs at one distance: integer series, repeated rows)
    const unsigned long long differ = st->kand ^ st->kor, all = st->kand;
    const bool equal = differ == 0ull;
    // leading bits that every key of the pass shares: past the digit where they all
    // lie in one bin, and the next digit starts behind them
    const int shared = equal ? 0 : __clzll((long long)differ);
    int shift, width;
    unsigned long long hi_mask;
    sel_digit(v.bits, shift, width, hi_mask);
    // thread t's bins t per .. t per + per - 1; exclusive prefix of the
    // per-thread sums within each wave by shuffles, then across the waves
    constexpr int per = 4096 / nt;
    unsigned long long sum = 0;
    for (int q = 0; q < per; ++q) sum += st->hist[t * per + q];
    unsigned long long incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(incl, o);
        if ((t & 63) >= o) incl += y;
    }
    if ((t & 63) == 63) sh.part[t >> 6] = incl;
    __syncthreads();
    unsigned long long before = incl - sum;
    for (int w = 0; w < (t >> 6); ++w) before += sh.part[w];
    const unsigned long long before0 = before;
    if (v.rank >= before && v.rank < before + sum) {   // one thread
        int bin = t * per;
        unsigned long long cnt = st->hist[bin];
        while (v.rank >= before + cnt) {
            before += cnt;
            cnt = st->hist[++bin];
        }
        unsigned long long p = v.prefix | ((unsigned long long)bin << shift);
        int bits = v.bits + width;
        if (shared > bits) {
            bits = shared;
            p = all & ~((1ull << (64 - shared)) - 1ull);
        }
        st->prefix = p;
        st->bits = bits;
        st->rank = v.rank - before;
        st->src = v.src;
        st->count = 0;
        if (equal) select_done(st, stats, v.base + all);
        else if (bits >= 64) select_done(st, stats, v.base + p);
        else st->mode = cnt <= (unsigned long long)kSelFew ? 1 : 0;
    }
    if (t == nt - 1 && v.rank >= before0 + sum) {
        // fewer keys than pairs: some distances are NaN
        select_done(st, stats, 0x7ff8000000000000ull);
    }
    __syncthreads();
    for (int q = t; q < 4096; q += nt) st->hist[q] = 0;
    if (t == 0) {
        st->kand = ~0ull;
        st->kor = 0ull;
    }
}

// Digit passes and the last collection by one workgroup of NT threads (at most 6
// digits resolve 64 bits), from the state as it stands.
template <int NT>
__device__ __forceinline__ void select_alone(const double *D2, int64_t ld, int64_t n, SelectState *st,
                                             SelView v, const unsigned long long *buf, double *stats,
                                             unsigned int *h, PickShared &sh) {
    for (int p = 0; p < 7 && v.mode != 2; ++p) {
        select_pass_body<NT>(D2, ld, n, 0, n, st, v, buf, 0, 1, h);
        __threadfence();
        __syncthreads();
        select_pick_body<NT>(st, v, stats, sh);
        __threadfence();
        __syncthreads();
        v = select_load(st);
    }
}

// One pass over the stored matrix or its bracket buffer with the pick by the
// last of its nb workgroups (the ticket counts them; every workgroup's
// histogram and candidates are published before its ticket).  kFinish: the last
// pass, whose last workgroup goes on alone if the answer is still not known.
template <bool kFinish>
__device__ __forceinline__ void select_pass_pick(const double *D2, int64_t ld, int64_t n,
                                                 SelectState *st, const unsigned long long *buf,
                                                 int64_t cap, bool gathered, bool first,
                                                 double *stats, int64_t b, int64_t nb) {
    __shared__ __align__(16) unsigned int h[4096];
    __shared__ PickShared sh;
    __shared__ int last;
    const SelView v = first ? select_start(st, n, cap, gathered) : select_load(st);
    if (v.mode == 2) {
        if (first && b == 0 && threadIdx.x == 0) select_done(st, stats, v.base + v.prefix);
        return;
    }
    select_pass_body<256>(D2, ld, n, 0, n, st, v, buf, b, nb, h);
    if (!last_workgroup(&st->ticket, (unsigned int)nb, &last)) return;
    select_pick_body<256>(st, v, stats, sh);
    if constexpr (kFinish) {
        __threadfence();
        __syncthreads();
        select_alone<256>(D2, ld, n, st, select_load(st), buf, stats, h, sh);
    }
}

template <bool kFinish>
__global__ __launch_bounds__(256) void k_select_pass(const double *D2, int64_t ld, int64_t n,
                                                     SelectState *st, const unsigned long long *buf,
                                                     int64_t cap, int gathered, int first,
                                                     double *stats) {
    select_pass_pick<kFinish>(D2, ld, n, st, buf, cap, gathered, first, stats, blockIdx.x, gridDim.x);
}

// The whole selection from the bracket buffer by one workgroup of 1024 threads,
// histogram and candidates in LDS: through the state in memory, as between
// launches, two passes with their fences took 26 us at n = 256, this takes 9.
__device__ __forceinline__ void select_buffer_alone(SelectState *st, const SelView &v,
                                                    const unsigned long long *buf, double *stats,
                                                    unsigned int *h, PickShared &sh) {
    __shared__ unsigned long long s_prefix, s_rank;
    __shared__ unsigned int s_left;
    const int t = threadIdx.x;
    const int64_t nk = (int64_t)st->nbuf;
    unsigned long long prefix = v.prefix, rank = v.rank;
    int64_t left = nk;   // keys under the prefix
    int bits = v.bits, shift, width;
    unsigned long long hi_mask;
    while (bits < 64 && left > kSelFew) {
        sel_digit(bits, shift, width, hi_mask);
        ((uint4 *)h)[t] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        for (int64_t q = t; q < nk; q += 1024) {
            const unsigned long long x = buf[q] - v.base;
            if ((x & hi_mask) == prefix) atomicAdd(&h[(x >> shift) & ((1ull << width) - 1ull)], 1u);
        }
        __syncthreads();
        // thread t's bins 4 t .. 4 t + 3 behind the bins of the threads before it
        const uint4 c = ((const uint4 *)h)[t];
        const unsigned int sum = c.x + c.y + c.z + c.w;
        unsigned int incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = __shfl_up(incl, o);
            if ((t & 63) >= o) incl += y;
        }
        if ((t & 63) == 63) sh.part[t >> 6] = incl;
        __syncthreads();
        unsigned long long before = incl - sum;
        for (int w = 0; w < (t >> 6); ++w) before += sh.part[w];
        if (rank >= before && rank < before + sum) {   // one thread
            const unsigned int cq[4] = {c.x, c.y, c.z, c.w};
            int q = 0;
            while (rank >= before + cq[q]) before += cq[q++];
            s_prefix = prefix | ((unsigned long long)(4 * t + q) << shift);
            s_rank = rank - before;
            s_left = cq[q];
        }
        __syncthreads();
        prefix = s_prefix;
        rank = s_rank;
        left = s_left;
        bits += width;
    }
    if (bits >= 64) {
        if (t == 0) {
            st->prefix = prefix;
            select_done(st, stats, v.base + prefix);
        }
        return;
    }
    sel_digit(bits, shift, width, hi_mask);
    __syncthreads();
    if (t == 0) s_left = 0;
    __syncthreads();
    for (int64_t q = t; q < nk; q += 1024) {
        const unsigned long long x = buf[q] - v.base;
        if ((x & hi_mask) == prefix) sh.keys[atomicAdd(&s_left, 1u)] = x;   // at most kSelFew
    }
    __syncthreads();
    const unsigned int cnt = s_left;
    if (t < (int)cnt) {
        const unsigned long long mine = sh.keys[t];
        unsigned int lt = 0, le = 0;
        for (unsigned int j = 0; j < cnt; ++j) {
            lt += sh.keys[j] < mine ? 1u : 0u;
            le += sh.keys[j] <= mine ? 1u : 0u;
        }
        if (lt <= rank && rank < le) {
            st->prefix = mine;
            select_done(st, stats, v.base + mine);
        }
    }
}

// The whole selection by one workgroup, for at most kSelSmall nodes.
__device__ __forceinline__ void select_small_body(const double *D2, int64_t ld, int64_t n,
                                                  SelectState *st, const unsigned long long *buf,
                                                  int64_t cap, bool gathered, double *stats) {
    __shared__ __align__(16) unsigned int h[4096];
    __shared__ PickShared sh;
    const SelView v = select_start(st, n, cap, gathered);
    if (v.mode == 2) {
        if (threadIdx.x == 0) select_done(st, stats, v.base + v.prefix);
        return;
    }
    if (v.src == 1) select_buffer_alone(st, v, buf, stats, h, sh);
    else select_alone<1024>(D2, ld, n, st, v, buf, stats, h, sh);
}

__global__ __launch_bounds__(1024) void k_select_small(const double *D2, int64_t ld, int64_t n,
                                                       SelectState *st, const unsigned long long *buf,
                                                       int64_t cap, int gathered, double *stats) {
    select_small_body(D2, ld, n, st, buf, cap, gathered, stats);
}

// Workgroups of a pass over n nodes.  With a bracket: 32 rows of the matrix each,
// and about 12 buffered keys a thread; 256 at most, since each adds its histogram
// to the same 4096 bins.  Over the whole matrix twice as many keep more loads in
// flight (seven passes at n = 4096 103 us, with 1024 workgroups 134, 128 163; at
// 16384 0.72 ms, 0.76, with 256 1.14).
static int select_grid(int64_t n, bool gathered) {
    const int64_t g = gathered ? n / 32 : n / 8, most = gathered ? 256 : 512;
    return (int)(g < 1 ? 1 : g < most ? g : most);
}

// Passes of the whole chip.  With a bracket the third digit leaves at most kSelFew
// distinct keys unless they crowd in one bin of 2^-36 of the bracket, the fourth
// pass ranks them, equal keys and leading bits that a crowd shares are found by
// AND and OR, and the last workgroup of the fourth finishes what is left (crowds
// within crowds).  Without one, and for matrices that a
// single workgroup could not read in time, as many passes as 64 bits need.
constexpr int kSelPasses = 4, kSelAllPasses = 7;
constexpr int64_t kSelFinishNodes = 20000;
static int select_passes(int64_t n, bool gathered) {
    return n <= kSelSmall ? 0 : n <= kSelFinishNodes && gathered ? kSelPasses : kSelAllPasses;
}

hipError_t launch_select_reset(SelectState *st, hipStream_t s) {
    hipLaunchKernelGGL(k_select_reset, dim3(1), dim3(256), 0, s, st);
    return hipGetLastError();
}

hipError_t launch_select_presample(const double *Xp, int64_t Tp, const double *sqn, int64_t n,
                                   SelectState *st, unsigned long long *buf, hipStream_t s) {
    if (select_buffer_keys(n) < kSelSample) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_select_sample_keys, dim3(kSelSample / 16), dim3(256), 0, s, Xp, Tp, sqn, n,
                       kSelSample, buf, st);
    hipLaunchKernelGGL(k_select_rank, dim3(kSelSample / 64), dim3(1024), 0, s, buf, kSelSample,
                       kSelMargin, n, sqn, Tp, st);
    return hipGetLastError();
}

hipError_t launch_select_median(const double *D2, int64_t ld, int64_t n, SelectState *st,
                                unsigned long long *buf, bool gathered, double *stats,
                                hipStream_t s) {
    const int64_t cap = select_buffer_keys(n);
    const int passes = select_passes(n, gathered);
    if (passes == 0) {
        hipLaunchKernelGGL(k_select_small, dim3(1), dim3(1024), 0, s, D2, ld, n, st, buf, cap,
                           gathered ? 1 : 0, stats);
        return hipGetLastError();
    }
    const dim3 grid(select_grid(n, gathered)), blk(256);
    for (int p = 0; p + 1 < passes; ++p)
        hipLaunchKernelGGL(k_select_pass<false>, grid, blk, 0, s, D2, ld, n, st, buf, cap, gathered ? 1 : 0,
                           p == 0 ? 1 : 0, stats);
    hipLaunchKernelGGL(k_select_pass<true>, grid, blk, 0, s, D2, ld, n, st, buf, cap, gathered ? 1 : 0, 0,
                       stats);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Streamed selection (no stored matrix): radix digits from the top bit, each
// digit one k_select_panel per recomputed row panel of the upper triangle and
// one pick; the collect pass and the final ranks are those of the stored path.

__global__ void k_select_start_top(SelectState *st, int64_t n) {
    if (threadIdx.x != 0) return;
    const unsigned long long N = (unsigned long long)n * (unsigned long long)(n - 1) / 2ull;
    st->rank = (N - 1ull) / 2ull;
    st->prefix = 0ull;
    st->bits = 0;
    st->mode = 0;
    st->src = 0;
    st->count = 0;
}

hipError_t launch_select_start_top(SelectState *st, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_select_reset, dim3(1), dim3(256), 0, s, st);
    hipLaunchKernelGGL(k_select_start_top, dim3(1), dim3(64), 0, s, st, n);
    return hipGetLastError();
}

// A panel's share of a digit (the pick follows the last panel).
__global__ __launch_bounds__(256) void k_select_panel(const double *D2, int64_t ld, int64_t n,
                                                      int64_t row0, int64_t row1,
                                                      SelectState *st) {
    __shared__ __align__(16) unsigned int h[4096];
    const SelView v = select_load(st);
    if (v.mode == 2) return;
    select_pass_body<256>(D2, ld, n, row0, row1, st, v, nullptr, blockIdx.x, gridDim.x, h);
}

__global__ __launch_bounds__(1024) void k_select_pick(SelectState *st, double *stats) {
    __shared__ PickShared sh;
    select_pick_body<1024>(st, select_load(st), stats, sh);
}

// One radix pass over the streamed bracket's buffer, with its pick.
__global__ __launch_bounds__(256) void k_select_buffer(SelectState *st, const unsigned long long *buf,
                                                       double *stats) {
    select_pass_pick<false>(nullptr, 0, 0, st, buf, 0, true, false, stats, blockIdx.x, gridDim.x);
}

hipError_t launch_select_panel(const double *D2p, int64_t ld, int64_t n, int64_t row0,
                               int64_t row1, SelectState *st, hipStream_t s) {
    if (row1 <= row0) return hipSuccess;
    const int64_t rows = row1 - row0;
    const int grid = (int)(rows < 2048 ? rows : 2048);
    hipLaunchKernelGGL(k_select_panel, dim3(grid), dim3(256), 0, s, D2p, ld, n, row0, row1, st);
    return hipGetLastError();
}

hipError_t launch_select_pick(SelectState *st, double *stats, hipStream_t s) {
    hipLaunchKernelGGL(k_select_pick, dim3(1), dim3(1024), 0, s, st, stats);
    return hipGetLastError();
}

// The streamed bracket: kStreamSample distances of pseudo-random pairs
// from the padded series (an estimate of the quantile only: the bracket is
// checked against exact counts), bracket of kStreamMargin sample ranks
// on each side of the target; then one sweep over the upper panels counts the
// keys below the bracket and gathers those inside it, and the radix passes run
// over the gathered keys.  The larger sample keeps the bracket to about 2.3 %
// of the keys.  Sample and ranks run on the whole chip (one workgroup, a
// thread per dot product and a sort in LDS took 6.0 ms at T = 360; 0.05 now).
constexpr int kStreamSample = 16384;
constexpr int kStreamMargin = 192;   // 3 sqrt(kStreamSample / 4)

int64_t select_stream_keys(int64_t n) {
    const int64_t N = n * (n - 1) / 2;
    return N / 100 * 3 + 65536;
}

hipError_t launch_select_sample_x(const double *Xp, int64_t Tp, const double *sqn, int64_t n,
                                  SelectState *st, unsigned long long *buf, hipStream_t s) {
    // (buf holds at least 65536 keys)
    hipLaunchKernelGGL(k_select_sample_keys, dim3(kStreamSample / 16), dim3(256), 0, s, Xp, Tp, sqn, n,
                       kStreamSample, buf, st);
    hipLaunchKernelGGL(k_select_rank, dim3(kStreamSample / 64), dim3(1024), 0, s, buf, kStreamSample,
                       kStreamMargin, n, sqn, Tp, st);
    return hipGetLastError();
}

hipError_t launch_select_bracket_panel(const double *D2p, int64_t ld, int64_t n, int64_t row0,
                                       int64_t row1, SelectState *st, unsigned long long *buf,
                                       int64_t cap, hipStream_t s) {
    if (row1 <= row0) return hipSuccess;
    const int64_t rows = row1 - row0;
    const int grid = (int)(rows < 2048 ? rows : 2048);
    hipLaunchKernelGGL(k_select_bracket_flush, dim3(grid), dim3(256), 0, s, D2p, ld, n, row0, row1,
                       st, buf, cap);
    return hipGetLastError();
}

hipError_t launch_select_check(SelectState *st, int64_t cap, double *stats, hipStream_t s) {
    hipLaunchKernelGGL(k_select_check, dim3(1), dim3(64), 0, s, st, cap, stats);
    return hipGetLastError();
}

hipError_t launch_select_buffer_pass(SelectState *st, const unsigned long long *buf, int64_t cap,
                                     double *stats, hipStream_t s) {
    // up to 2^24 keys 512 workgroups at most, as for stored snapshots; the
    // billions of a larger one need the whole chip's bandwidth
    const int64_t most = cap <= ((int64_t)1 << 24) ? 512 : 2048;
    const int grid = (int)(cap / 2048 + 1 < most ? cap / 2048 + 1 : most);
    hipLaunchKernelGGL(k_select_buffer, dim3(grid), dim3(256), 0, s, st, buf, stats);
    return hipGetLastError();
}

// Row panel of the weights from its squared distances, in place: W_ij =
// exp(-D2_ij / sigma^2) for i != j (both < n), else 0 - the expression of
// k_exp_sym, so each value equals the stored matrix's bit for bit.  Panel row
// q is node row0 + q.  deg != nullptr: deg_i = sum_j W_ij (fixed order).
// dinv != nullptr: fro[q] = sum_j (W_ij dinv_i dinv_j)^2 with dinv = D^{-1/2},
// a row of the squared Frobenius norm of S = D^{-1/2} W D^{-1/2}.
__global__ __launch_bounds__(256) void k_exp_rows(double *Wp, int64_t ld, int64_t n,
                                                  int64_t row0, const double *stats,
                                                  double *deg, const double *dinv,
                                                  double *fro) {
    __shared__ double red[4];
    const int64_t i = row0 + blockIdx.x;
    double *row = Wp + (int64_t)blockIdx.x * ld;
    const double sigma = stats[1];
    const double s2 = sigma * sigma;
    const bool live = i < n;
    const double di = (dinv && live) ? dinv[i] : 0.0;
    double acc = 0.0, f = 0.0;
    for (int64_t j0 = threadIdx.x; j0 < ld; j0 += 4 * 256) {
        double d2[4];   // four loads in flight before the first exp
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = j0 + 256 * u;
            d2[u] = j < ld ? row[j] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = j0 + 256 * u;
            if (j >= ld) break;
            const double v = (live && j < n && i != j) ? exp(-d2[u] / s2) : 0.0;
            row[j] = v;
            acc += v;
            if (dinv && v != 0.0) {
                const double sv = v * di * dinv[j];
                f += sv * sv;
            }
        }
    }
    acc = block_sum256(acc, red);
    if (deg && live && threadIdx.x == 0) deg[i] = acc;
    if (fro) {
        f = block_sum256(f, red);
        if (threadIdx.x == 0) fro[blockIdx.x] = f;
    }
}

hipError_t launch_exp_rows(double *Wp, int64_t ld, int64_t n, int64_t row0, int64_t rows,
                           const double *stats, double *deg, const double *dinv, double *fro,
                           hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_exp_rows, dim3((unsigned)rows), dim3(256), 0, s, Wp, ld, n, row0, stats,
                       deg, dinv, fro);
    return hipGetLastError();
}

__global__ void k_set_sigma(double sigma, double *stats) { stats[1] = sigma; }

hipError_t launch_set_sigma(double sigma, double *stats, hipStream_t s) {
    hipLaunchKernelGGL(k_set_sigma, dim3(1), dim3(1), 0, s, sigma, stats);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------

int sym_tiles64(int64_t ld) {
    const int nt = (int)(ld / 64);
    return nt * (nt + 1) / 2;
}

// One 64 x 64 tile (I <= J) per workgroup.  part[J][i] receives the sum of
// row i over the tile's columns and, for I < J, part[I][j] the sum of column
// j: every (tile column, node) slot is written by exactly one tile.  A lane
// takes two adjacent columns of every other row (16-byte loads and stores),
// so a wave access covers two contiguous 512-byte row segments; the four
// waves take 16 rows each.  The mirror is written from the LDS copy, two
// adjacent rows per lane.
// Upper tile `id` (after the XCD remap) of the sym_tile<8> order.
__device__ __forceinline__ void exp_sym_tile(double *W, int64_t ld, int64_t n,
                                             const double *stats, int nt, double *part, int id) {
    struct alignas(16) D2 { double x, y; };
    __shared__ double t[64][66];   // even pitch: 16-byte rows of pairs
    __shared__ double cs[4][64];
    int I, J;
    sym_tile<8>(id, nt, I, J);
    const double sigma = stats[1];
    const double s2 = sigma * sigma;
    const int64_t i0 = (int64_t)I * 64, j0 = (int64_t)J * 64;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int cp = lane & 31, h = lane >> 5;
    const int64_t ja = j0 + 2 * cp;   // this lane's columns ja, ja + 1
    double c0 = 0.0, c1 = 0.0;
    D2 d2[8];   // all eight row loads in flight before the first exp
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) d2[rr] = *(const D2 *)(W + (i0 + wv * 16 + 2 * rr + h) * ld + ja);
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
        const int r = wv * 16 + 2 * rr + h;
        const int64_t i = i0 + r;
        D2 v;
        v.x = (i < n && ja < n && i != ja) ? exp(-d2[rr].x / s2) : 0.0;
        v.y = (i < n && ja + 1 < n && i != ja + 1) ? exp(-d2[rr].y / s2) : 0.0;
        *(D2 *)(W + i * ld + ja) = v;
        *(D2 *)&t[r][2 * cp] = v;
        c0 += v.x;
        c1 += v.y;
    }
    // this wave's column sums: the two halves hold the even and odd rows
    c0 += __shfl_xor(c0, 32);
    c1 += __shfl_xor(c1, 32);
    if (h == 0) {
        cs[wv][2 * cp] = c0;
        cs[wv][2 * cp + 1] = c1;
    }
    __syncthreads();
    {   // row sums: thread (row r, quarter q) over 16 columns
        const int r = threadIdx.x >> 2, q = threadIdx.x & 3;
        double rs = 0.0;
#pragma unroll
        for (int c = 0; c < 16; ++c) rs += t[r][16 * q + c];
        rs += __shfl_xor(rs, 1);
        rs += __shfl_xor(rs, 2);
        if (q == 0) part[(int64_t)J * ld + i0 + r] = rs;
    }
    if (I == J) return;
    if (threadIdx.x < 64)
        part[(int64_t)I * ld + j0 + threadIdx.x] =
            (cs[0][threadIdx.x] + cs[1][threadIdx.x]) + (cs[2][threadIdx.x] + cs[3][threadIdx.x]);
#pragma unroll 4
    for (int cc = 0; cc < 8; ++cc) {   // mirror: row j0 + c gets column c of the tile
        const int c = wv * 16 + 2 * cc + h;
        const D2 m{t[2 * cp][c], t[2 * cp + 1][c]};
        *(D2 *)(W + (j0 + c) * ld + i0 + 2 * cp) = m;
    }
}

__global__ __launch_bounds__(256) void k_exp_sym(double *W, int64_t ld, int64_t n,
                                                 const double *stats, int nt, double *part) {
    exp_sym_tile(W, ld, n, stats, nt, part, xcd_remap(blockIdx.x, nt * (nt + 1) / 2));
}

// Degrees of 64 nodes from the tile columns' partials: four threads per node
// sum a quarter of the tiles each, in order, 32 loads in flight; the quarters
// are added in order.
__device__ __forceinline__ void degree_body(const double *part, int nt, int64_t ld, int64_t n,
                                            double *deg, int64_t b, double (*sq)[64]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t i = b * 64 + lane;
    const int q0 = w * nt / 4, q1 = (w + 1) * nt / 4;
    sq[w][lane] = i < n ? ordered_sum(part + (int64_t)q0 * ld + i, ld, q1 - q0, 0.0) : 0.0;
    __syncthreads();
    if (w == 0 && i < n) deg[i] = (sq[0][lane] + sq[1][lane]) + (sq[2][lane] + sq[3][lane]);
}

__device__ __forceinline__ void graph_stats_body(const double *deg, int64_t n, double *stats,
                                                 double *red) {
    double s = 0.0, lo = INFINITY, hi = -INFINITY;
    // a thread's nodes in increasing order, sixteen loads in flight
    for (int64_t i0 = threadIdx.x; i0 < n; i0 += 16 * 256) {
        double dv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) dv[u] = i0 + 256 * u < n ? deg[i0 + 256 * u] : 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            if (i0 + 256 * u >= n) break;
            const double d = dv[u];
            s += d;
            // a NaN stays: it is the smallest and the largest from then on
            lo = isnan(lo) || isnan(d) ? NAN : fmin(lo, d);
            hi = isnan(hi) || isnan(d) ? NAN : fmax(hi, d);
        }
    }
    s = block_sum256(s, red);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const double a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
        lo = isnan(lo) || isnan(a) ? NAN : fmin(lo, a);
        hi = isnan(hi) || isnan(b) ? NAN : fmax(hi, b);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = lo;
        red[4 + (threadIdx.x >> 6)] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) {
            lo = isnan(lo) || isnan(red[w]) ? NAN : fmin(lo, red[w]);
            hi = isnan(hi) || isnan(red[4 + w]) ? NAN : fmax(hi, red[4 + w]);
        }
        stats[0] = s;
        stats[2] = lo;
        stats[3] = hi;
    }
}

// The degrees, then the statistics by the last of nb workgroups (the degrees
// are published before a workgroup's ticket).
__device__ __forceinline__ void degree_stats(const double *part, int nt, int64_t ld, int64_t n,
                                             double *deg, double *stats, int *ticket, int64_t b,
                                             int64_t nb) {
    __shared__ double sq[4][64], red[8];
    __shared__ int last;
    degree_body(part, nt, ld, n, deg, b, sq);
    if (!last_workgroup((unsigned int *)ticket, (unsigned int)nb, &last)) return;
    graph_stats_body(deg, n, stats, red);
}

__global__ __launch_bounds__(256) void k_degree_stats(const double *part, int nt, int64_t ld,
                                                      int64_t n, double *deg, double *stats,
                                                      int *ticket) {
    degree_stats(part, nt, ld, n, deg, stats, ticket, blockIdx.x, gridDim.x);
}

hipError_t launch_exp_degree(double *W, int64_t ld, int64_t n, double *stats, double *deg,
                             double *part, int *ticket, hipStream_t s) {
    const int nt = (int)(ld / 64);
    hipLaunchKernelGGL(k_exp_sym, dim3((unsigned)sym_tiles64(ld)), dim3(256), 0, s, W, ld, n,
                       (const double *)stats, nt, part);
    hipLaunchKernelGGL(k_degree_stats, dim3((unsigned)cdiv(n, 64)), dim3(256), 0, s, part, nt, ld, n,
                       deg, stats, ticket);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_graph_stats(const double *deg, int64_t n,
                                                     double *stats) {
    __shared__ double red[8];
    graph_stats_body(deg, n, stats, red);
}

hipError_t launch_graph_stats(const double *deg, int64_t n, double *stats, hipStream_t s) {
    hipLaunchKernelGGL(k_graph_stats, dim3(1), dim3(256), 0, s, deg, n, stats);
    return hipGetLastError();
}

// Caller-supplied weights: copy into the padded layout, zero the diagonal,
// row sums, and flag non-finite (1), negative (2) or asymmetric (4) input.
__global__ __launch_bounds__(256) void k_import_weights(const double *Win, int64_t ldw,
                                                        int64_t n, double *W, int64_t ld,
                                                        double *deg, int *flags) {
    __shared__ double red[4];
    const int64_t i = blockIdx.x;
    double s = 0.0;
    int f = 0;
    for (int64_t j = threadIdx.x; j < ld; j += 256) {
        double v = 0.0;
        if (i < n && j < n && i != j) {
            v = Win[i * ldw + j];
            if (!isfinite(v)) f |= 1;
            if (v < 0.0) f |= 2;
            if (v != Win[j * ldw + i]) f |= 4;
        }
        W[i * ld + j] = v;
        s += v;
    }
    s = block_sum256(s, red);
    if (threadIdx.x == 0 && i < n) deg[i] = s;
    if (f) atomicOr(flags, f);
}

hipError_t launch_import_weights(const double *Win, int64_t ldw, int64_t n, double *W,
                                 int64_t ld, double *deg, int *flags, hipStream_t s) {
    hipLaunchKernelGGL(k_import_weights, dim3((unsigned)ld), dim3(256), 0, s, Win, ldw, n, W,
                       ld, deg, flags);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The graph build of many snapshots in grouped launches: each kernel below
// runs, for workgroup blockIdx.x, the per-snapshot kernel's workgroup
// blockIdx.x - prefix[p] of snapshot p (found through the kernel's prefix
// table), with that snapshot's arguments, so the results are the
// per-snapshot kernels' bit for bit.

bool select_uses_bracket(int64_t n, bool allowed) {
    const double N = (double)n * (double)(n - 1) / 2.0;
    return allowed && N * 2.0 * kSelMargin / kSelSample <= 0.8 * (double)select_buffer_keys(n);
}

int graph_gram_shape(int P, const int64_t *ld, const int64_t *T) {
    for (int t = 0; t < P; ++t)
        if (pad_t(T[t]) >= kGramFar) return 2;
    int64_t c0 = 0, c1 = 0;
    for (int t = 0; t < P; ++t) {
        c0 += gram_wgs(0, kGramUpper, ld[t], 0, ld[t]);
        c1 += gram_wgs(1, kGramUpper, ld[t], 0, ld[t]);
    }
    return (double)cdiv(c1, 256) / 0.8 < 4.0 * (double)cdiv(c0, 256) ? 1 : 0;
}

int graph_table_count(int tb, int64_t n, int64_t ld, bool bracket, int gram_shape) {
    switch (tb) {
    case kGtRows: return (int)(ld / 4);
    case kGtOne: return 1;
    case kGtGram: return (int)gram_wgs(gram_shape, kGramUpper, ld, 0, ld);
    case kGtSample: return bracket ? kSelSample / 64 : 0;
    case kGtPass: return select_grid(n, bracket);
    case kGtSym: return sym_tiles64(ld);
    case kGtNodes64: return (int)cdiv(n, 64);
    case kGtPrep: return (int)cdiv(ld, 256);
    default: return 0;
    }
}

struct GroupSlot {
    int p;
    int64_t b, nb;
};
__device__ __forceinline__ GroupSlot group_slot(const int *prefix, int P) {
    GroupSlot g;
    g.p = group_find(prefix, P, blockIdx.x);
    g.b = blockIdx.x - prefix[g.p];
    g.nb = prefix[g.p + 1] - prefix[g.p];
    return g;
}

__global__ __launch_bounds__(256) void k_graph_init_grouped(const GraphSnap *snaps, const int *prefix,
                                                            int P, int select) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    if (threadIdx.x < 64) d.flags[threadIdx.x] = 0;
    if (select) {
        select_reset_body(d.sel);
        select_bracket_reset(d.sel);
    }
}

__global__ __launch_bounds__(256) void k_pad_grouped(const GraphSnap *snaps, const int *prefix, int P) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    pad_row(d.X, d.n, d.T, d.ldx, d.Xp, d.Tp, d.sqn, nullptr, g.b * 4 + (threadIdx.x >> 6));
}

__global__ __launch_bounds__(256) void k_select_keys_grouped(const GraphSnap *snaps, const int *prefix,
                                                             int P) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    select_sample_keys_body(d.Xp, d.Tp, d.sqn, d.n, kSelSample, d.buf,
                            (int)g.b * 4 + (threadIdx.x >> 6), (int)g.nb * 4);
}

__global__ __launch_bounds__(1024) void k_select_rank_grouped(const GraphSnap *snaps, const int *prefix,
                                                             int P) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    select_rank_body(d.buf, kSelSample, kSelMargin, d.n, d.sqn, d.Tp, d.sel, (int)g.b);
}

template <int SHAPE>
__global__ __launch_bounds__(GramCfg<SHAPE>::Core::NT, GramCfg<SHAPE>::WAVES) void k_gram_grouped(
    const GraphSnap *snaps, const int *prefix, int P, int select) {
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    gram_tile<SHAPE, false, false>(d.Xp, d.Tp, d.sqn, d.n, d.ld, d.W, 0, d.ld, kGramUpper,
                            xcd_remap((int)g.b, (int)g.nb), select ? d.sel : nullptr,
                            (const double *)nullptr, (double *)smem_raw,
                            select && d.bracket ? d.buf : nullptr, d.cap);
}

template <int SHAPE>
static hipError_t gram_grouped_launch(const GraphSnap *snaps, const int *prefix, int total, int P,
                                      int select, hipStream_t s) {
    using Core = typename GramCfg<SHAPE>::Core;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void *)k_gram_grouped<SHAPE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)Core::SMEM);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL(k_gram_grouped<SHAPE>, dim3(total), dim3(Core::NT), Core::SMEM, s, snaps, prefix,
                       P, select);
    return hipGetLastError();
}

template <bool kFinish>
__global__ __launch_bounds__(256) void k_select_pass_grouped(const GraphSnap *snaps, const int *prefix,
                                                             int P, int first) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    select_pass_pick<kFinish>(d.W, d.ld, d.n, d.sel, d.buf, d.cap, d.bracket != 0, first != 0, d.stats, g.b,
                              g.nb);
}

__global__ __launch_bounds__(1024) void k_select_small_grouped(const GraphSnap *snaps, const int *prefix,
                                                               int P) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    select_small_body(d.W, d.ld, d.n, d.sel, d.buf, d.cap, d.bracket != 0, d.stats);
}

__global__ void k_set_sigma_grouped(const GraphSnap *snaps, const int *prefix, int P, double sigma) {
    const GroupSlot g = group_slot(prefix, P);
    if (threadIdx.x == 0) snaps[g.p].stats[1] = sigma;
}

__global__ __launch_bounds__(256) void k_exp_sym_grouped(const GraphSnap *snaps, const int *prefix, int P) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    const int nt = (int)(d.ld / 64);
    exp_sym_tile(d.W, d.ld, d.n, d.stats, nt, d.dpart, xcd_remap((int)g.b, (int)g.nb));
}

__global__ __launch_bounds__(256) void k_degree_stats_grouped(const GraphSnap *snaps, const int *prefix,
                                                              int P) {
    const GroupSlot g = group_slot(prefix, P);
    const GraphSnap &d = snaps[g.p];
    degree_stats(d.dpart, (int)(d.ld / 64), d.ld, d.n, d.deg, d.stats, d.flags + kDegreeTicket, g.b, g.nb);
}

hipError_t launch_graph_grouped(const GraphSnap *snaps, const int *tables, const int *totals,
                                int P, int64_t nmax, double sigma, int gram_shape, hipStream_t s) {
    auto tb = [&](int t) { return tables + (size_t)t * (P + 1); };
    const bool select = sigma <= 0.0;
    hipLaunchKernelGGL(k_graph_init_grouped, dim3(totals[kGtOne]), dim3(256), 0, s, snaps, tb(kGtOne), P,
                       select ? 1 : 0);
    hipLaunchKernelGGL(k_pad_grouped, dim3(totals[kGtRows]), dim3(256), 0, s, snaps, tb(kGtRows), P);
    // the brackets from samples of the series; the Gram counts and gathers them
    if (select && totals[kGtSample] > 0) {
        hipLaunchKernelGGL(k_select_keys_grouped, dim3(totals[kGtSample]), dim3(256), 0, s, snaps,
                           tb(kGtSample), P);
        hipLaunchKernelGGL(k_select_rank_grouped, dim3(totals[kGtSample]), dim3(1024), 0, s, snaps,
                           tb(kGtSample), P);
    }
    hipError_t e;
    switch (gram_shape) {
    case 0: e = gram_grouped_launch<0>(snaps, tb(kGtGram), totals[kGtGram], P, select ? 1 : 0, s); break;
    case 1: e = gram_grouped_launch<1>(snaps, tb(kGtGram), totals[kGtGram], P, select ? 1 : 0, s); break;
    default: e = gram_grouped_launch<2>(snaps, tb(kGtGram), totals[kGtGram], P, select ? 1 : 0, s); break;
    }
    if (e != hipSuccess) return e;
    if (select) {
        // the passes that the largest snapshot takes (one of few enough nodes for
        // kSelPasses has a bracket whenever another has)
        const int passes = select_passes(nmax, totals[kGtSample] > 0);
        for (int q = 0; q + 1 < passes; ++q)
            hipLaunchKernelGGL(k_select_pass_grouped<false>, dim3(totals[kGtPass]), dim3(256), 0, s, snaps,
                               tb(kGtPass), P, q == 0 ? 1 : 0);
        if (passes > 0)
            hipLaunchKernelGGL(k_select_pass_grouped<true>, dim3(totals[kGtPass]), dim3(256), 0, s, snaps,
                               tb(kGtPass), P, 0);
        else
            hipLaunchKernelGGL(k_select_small_grouped, dim3(totals[kGtOne]), dim3(1024), 0, s, snaps,
                               tb(kGtOne), P);
    } else {
        hipLaunchKernelGGL(k_set_sigma_grouped, dim3(totals[kGtOne]), dim3(64), 0, s, snaps, tb(kGtOne), P,
                           sigma);
    }
    hipLaunchKernelGGL(k_exp_sym_grouped, dim3(totals[kGtSym]), dim3(256), 0, s, snaps, tb(kGtSym), P);
    hipLaunchKernelGGL(k_degree_stats_grouped, dim3(totals[kGtNodes64]), dim3(256), 0, s, snaps,
                       tb(kGtNodes64), P);
    return hipGetLastError();
}

} // namespace cdl
