// LDS-tiled MFMA cores for C = A * B^T (both operands row-major along the
// reduction index k), used by every dense contraction of the path.  Callers
// supply padded operands (K a multiple of BK, tile rows inside the
// allocation), so the cores have no bounds checks.  Operands go straight from
// global memory into LDS: RowCore for FP64 and FP32, DmaCore for 16-bit levels.
#pragma once

#include "common.h"

namespace cdl {

// Stage the BM x BN tile of values f(row, col, acc) (tile-local row, col) of
// type O in LDS (row stride BN + 16/sizeof(O)), then copy it to global
// memory as rows C + (m0 + r) * ldc + n0 and, if `mirror`, as its transpose
// C + (n0 + c) * ldc + m0.  `sC` must hold BM * (BN + 16/sizeof(O)) elements
// and may alias the core's operand stages (a barrier separates the uses).
// Every thread of the workgroup must call this.
template <class Core, typename O, class F>
__device__ inline void stage_and_store(Core &g, O *sC, F f, O *C, int64_t ldc,
                                       int64_t m0, int64_t n0, bool mirror) {
    constexpr int BM = Core::TBM, BN = Core::TBN, NT = Core::NT;
    constexpr int CEo = 16 / (int)sizeof(O);
    constexpr int LDC = BN + CEo;
    __syncthreads();
    if (!Core::half()) {
#pragma unroll
        for (int i = 0; i < Core::WTM; ++i)
#pragma unroll
            for (int j = 0; j < Core::WTN; ++j)
#pragma unroll
                for (int r = 0; r < Core::MF::R; ++r) {
                    int row = Core::row_of(i, r), col = Core::col_of(j);
                    sC[row * LDC + col] = f(row, col, g.acc[i][j][r]);
                }
    }
    __syncthreads();
    constexpr int CPR = BN / CEo;
    for (int ch = threadIdx.x; ch < BM * CPR; ch += NT) {
        int r = ch / CPR, c = ch % CPR;
        *(uint4 *)(C + (m0 + r) * ldc + n0 + c * CEo) = *(const uint4 *)(sC + r * LDC + c * CEo);
    }
    if (mirror) {
        constexpr int QPR = BM / CEo;
        for (int ch = threadIdx.x; ch < BN * QPR; ch += NT) {
            int c = ch % BN, q = ch / BN;
            union { uint4 v; O e[CEo]; } u;
#pragma unroll
            for (int e = 0; e < CEo; ++e) u.e[e] = sC[(q * CEo + e) * LDC + c];
            *(uint4 *)(C + (n0 + c) * ldc + m0 + q * CEo) = u.v;
        }
    }
}

// As stage_and_store for a 256 x 256 tile of 16-bit values f(row, col, acc),
// through a transposed copy in LDS without padding (128 KB): a lane's four
// consecutive rows of a column go out as one 8-byte write, the mirrored rows are
// read back as they lie, and the rows of the tile as 4 x 8 blocks that v_perm
// transposes.  The 16-byte chunks of a column are XOR-swizzled so that no access
// meets more lanes on a bank than its width needs.  With one value per LDS access
// and uncoalesced mirror rows the epilogue took about 40 us of a tile's 275 at n =
// 8192; 512 tiles there went from 551-595 to 450 us.
__device__ inline uint32_t tile16_place(int col, int chunk) {
    return (uint32_t)(col * 512 + 16 * (chunk ^ ((col ^ (col >> 3)) & 31)));
}
template <class Core, typename O, class F>
__device__ inline void stage_and_store16(Core &g, char *sT, F f, O *C, int64_t ldc, int64_t m0,
                                         int64_t n0, bool mirror) {
    constexpr int NT = Core::NT;
    static_assert(sizeof(O) == 2 && Core::TBM == 256 && Core::TBN == 256, "16-bit tiles of 256");
    using MF = typename Core::MF;
    static_assert(MF::R % 4 == 0, "rows in fours");
    __syncthreads();
    // the lane afresh, so that nothing of it lives in registers through the k loop
    int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row_w = wave % Core::NWM * Core::WTM * MF::M, col_w = wave / Core::NWM * Core::WTN * MF::M;
#pragma unroll
    for (int i = 0; i < Core::WTM; ++i)
#pragma unroll
        for (int j = 0; j < Core::WTN; ++j)
#pragma unroll
            for (int r = 0; r < MF::R; r += 4) {
                const int row = row_w + i * MF::M + MF::crow(lane, r), col = col_w + j * MF::M + MF::ccol(lane);
                union { uint2 v; O e[4]; } u;
#pragma unroll
                for (int q = 0; q < 4; ++q) u.e[q] = f(row + q, col, g.acc[i][j][r + q]);
                *(uint2 *)(sT + tile16_place(col, row >> 3) + 2 * (row & 4)) = u.v;
                __builtin_amdgcn_sched_barrier(0);   // one group at a time in registers
            }
    __syncthreads();
#pragma unroll 1
    for (int b = wave * 64 + lane; b < 2048; b += NT) {
        const int c8 = b & 31, rq = b >> 5;
        uint2 v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = *(const uint2 *)(sT + tile16_place(8 * c8 + e, rq >> 1) + 8 * (rq & 1));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t sel = r & 1 ? 0x07060302u : 0x05040100u;
            auto pair = [&](int e) {
                return r < 2 ? __builtin_amdgcn_perm(v[e + 1].x, v[e].x, sel)
                             : __builtin_amdgcn_perm(v[e + 1].y, v[e].y, sel);
            };
            *(uint4 *)(C + (m0 + 4 * rq + r) * ldc + n0 + 8 * c8) =
                make_uint4(pair(0), pair(2), pair(4), pair(6));
        }
    }
    if (mirror) {
#pragma unroll 4
        for (int b = wave * 64 + lane; b < 8192; b += NT) {
            const int c = b >> 5, q = b & 31;
            *(uint4 *)(C + (n0 + c) * ldc + m0 + 8 * q) = *(const uint4 *)(sT + tile16_place(c, q));
        }
    }
}

// As stage_and_store, staging RC rows of the tile at a time so that the
// staging buffer (RC * (BN + 16/sizeof(O)) elements) stays small.
template <int RC, class Core, typename O, class F>
__device__ inline void stage_and_store_rows(Core &g, O *sC, F f, O *C, int64_t ldc, int64_t m0,
                                            int64_t n0, bool mirror) {
    constexpr int BM = Core::TBM, BN = Core::TBN, NT = Core::NT;
    constexpr int CEo = 16 / (int)sizeof(O);
    constexpr int LDC = BN + CEo;
    static_assert(BM % RC == 0 && RC % CEo == 0, "bad row chunk");
#pragma unroll 1
    for (int r0 = 0; r0 < BM; r0 += RC) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < Core::WTM; ++i)
#pragma unroll
            for (int j = 0; j < Core::WTN; ++j)
#pragma unroll
                for (int r = 0; r < Core::MF::R; ++r) {
                    const int row = Core::row_of(i, r), col = Core::col_of(j);
                    if (row >= r0 && row < r0 + RC) sC[(row - r0) * LDC + col] = f(row, col, g.acc[i][j][r]);
                }
        __syncthreads();
        constexpr int CPR = BN / CEo;
        for (int ch = threadIdx.x; ch < RC * CPR; ch += NT) {
            const int r = ch / CPR, c = ch % CPR;
            *(uint4 *)(C + (m0 + r0 + r) * ldc + n0 + c * CEo) = *(const uint4 *)(sC + r * LDC + c * CEo);
        }
        if (mirror) {
            constexpr int QPR = RC / CEo;
            for (int ch = threadIdx.x; ch < BN * QPR; ch += NT) {
                const int c = ch % BN, q = ch / BN;
                union { uint4 v; O e[CEo]; } u;
#pragma unroll
                for (int e = 0; e < CEo; ++e) u.e[e] = sC[(q * CEo + e) * LDC + c];
                *(uint4 *)(C + (n0 + c) * ldc + m0 + r0 + q * CEo) = u.v;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// 16-bit operand core fed by direct global->LDS loads (gfx950
// buffer_load_dwordx4 ... lds): each wave instruction moves 64 x 16 bytes
// into 1 KB of LDS, so operands never pass through VGPRs.  The two operand
// panels are addressed through buffer resources (base = first row of the
// panel, in SGPRs); per instruction the wave-uniform part of the offset (row
// block, k-slice) is a scalar offset and the per-lane part one of two VGPR
// offsets, so the loads need no 64-bit address arithmetic.  LDS rows are
// BK = 64 elements (128 B) with the 16-byte chunks XOR-swizzled by
// (row >> 1) & 7, which keeps the 16 lanes that an ds_read_b128 serves per
// cycle on distinct banks for the 32-row MFMA fragments.
//
// Pipeline (two LDS stages): the fragments of k-step q + 1 are read while
// the MFMAs of k-step q run (sched_group_barrier interleaves one LDS read
// with the MFMAs that fit beside it); before the last k-step of a stage
// every wave waits for the next stage's loads and for its own last reads (without
// the latter another wave's loads could overtake them; it costs a third of a
// percent of a squaring at n = 8192) and meets the others at a barrier, then reads
// the next stage's first fragments beside the last k-step's MFMAs and issues the
// loads of the stage after next into the buffer
// just released.  The loop body is uniform; the last stage is peeled.

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;

template <int N> __device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The same, and every LDS read of this wave has returned.
template <int N> __device__ inline void wait_vmcnt_lds() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// Workgroup barrier without a memory fence (the loads into LDS are waited
// for explicitly); the empty asm statements keep the compiler from moving
// memory accesses across it.
__device__ inline void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <class Mf, int BM, int BN, int WM, int WN>
struct DmaCore {
    using T = typename Mf::T;
    using Frag = typename Mf::Frag;
    using AccV = typename Mf::AccV;
    using MF = Mf;
    static_assert(sizeof(T) == 2, "16-bit operands");
    static constexpr int BK = 64;
    static constexpr int TBM = BM, TBN = BN;
    static constexpr int NW = WM * WN, NT = NW * 64;
    static constexpr int CE = 8;                  // elements per 16-byte chunk
    static constexpr int CPR = BK / CE;           // 8 chunks per LDS row
    static constexpr int RPI = 64 / CPR;          // rows per wave instruction
    static constexpr int ROWB = BK * 2;           // bytes per LDS row
    static constexpr int STAGE = (BM + BN) * ROWB;
    static constexpr size_t SMEM = 2 * (size_t)STAGE;
    static constexpr int NWM = WM;
    static constexpr int WTM = BM / WM / Mf::M, WTN = BN / WN / Mf::M;
    static constexpr int AI = BM / RPI / NW, BI = BN / RPI / NW;
    static constexpr int NKK = BK / Mf::KI;
    static constexpr int NF = WTM + WTN;          // fragment reads per k-step
    static constexpr int NM = WTM * WTN;          // MFMAs per k-step
    static_assert(AI * RPI * NW == BM && BI * RPI * NW == BN, "rows per wave");
    static_assert(NKK >= 2 && NKK % 2 == 0, "an even number of k-steps per stage");

    AccV acc[WTM][WTN];

    __device__ static inline int swz(int c, int row) { return c ^ ((row >> 1) & 7); }

    // Loads of one 64-wide k-slice (element offset k0) of both panels into
    // the LDS stage at byte offset `stage`.  Row r of a panel lies at byte
    // r * ld * 2 of its resource; rows of one instruction start at a multiple
    // of 8, so their swizzle depends only on the parity of the row block.
    __device__ inline void issue(uint32_t stage, __amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb,
                                 int64_t lda, int64_t ldb, int64_t k0, int w, const uint32_t *voa,
                                 const uint32_t *vob) {
#pragma unroll
        for (int q = 0; q < AI; ++q) {
            const int blk = w * AI + q, row0 = blk * RPI;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                ra, (lds_void *)(uintptr_t)(stage + row0 * ROWB), 16, voa[blk & 1],
                (uint32_t)((int64_t)row0 * lda * 2 + k0 * 2), 0, 0);
        }
#pragma unroll
        for (int q = 0; q < BI; ++q) {
            const int blk = w * BI + q, row0 = blk * RPI;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rb, (lds_void *)(uintptr_t)(stage + (BM + row0) * ROWB), 16, vob[blk & 1],
                (uint32_t)((int64_t)row0 * ldb * 2 + k0 * 2), 0, 0);
        }
    }

    __device__ inline void load_frags(const char *s, int kk, Frag *f) {
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        const int wm = wid % WM, wn = wid / WM;
        const int ch = (kk + Mf::E * (lane / Mf::M)) / CE;
        const char *sA = s, *sB = s + BM * ROWB;
#pragma unroll
        for (int i = 0; i < WTM; ++i) {
            const int row = wm * WTM * Mf::M + i * Mf::M + lane % Mf::M;
            f[i] = *(const Frag *)(sA + row * ROWB + 16 * swz(ch, row));
        }
#pragma unroll
        for (int j = 0; j < WTN; ++j) {
            const int row = wn * WTN * Mf::M + j * Mf::M + lane % Mf::M;
            f[WTM + j] = *(const Frag *)(sB + row * ROWB + 16 * swz(ch, row));
        }
    }

    __device__ inline void mmas(const Frag *f) {
#pragma unroll
        for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int j = 0; j < WTN; ++j) acc[i][j] = Mf::mma(f[i], f[WTM + j], acc[i][j]);
    }

    // Scheduling order of one k-step: the NF fragment reads spread evenly
    // between its NM MFMAs.
    template <int I = 0> __device__ static inline void interleave() {
        constexpr int G = NF > NM ? NF : NM;
        constexpr int nd = (I + 1) * NF / G - I * NF / G;
        constexpr int nm = (I + 1) * NM / G - I * NM / G;
        if constexpr (nd > 0) __builtin_amdgcn_sched_group_barrier(0x100, nd, 0);
        if constexpr (nm > 0) __builtin_amdgcn_sched_group_barrier(0x008, nm, 0);
        if constexpr (I + 1 < G) interleave<I + 1>();
    }

    // Full K loop (K a multiple of 64; rows m0.. and n0.. of the operands
    // inside the allocations).  smem holds SMEM bytes.
    __device__ inline void run(const T *A, int64_t lda, const T *B, int64_t ldb, int64_t m0,
                               int64_t n0, int64_t K, void *smem_v) {
        char *smem = (char *)smem_v;
#pragma unroll
        for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int j = 0; j < WTN; ++j)
#pragma unroll
                for (int r = 0; r < Mf::R; ++r) acc[i][j][r] = 0;
        const int nk = (int)(K / BK);
        if (nk == 0) return;
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t s0 = (uint32_t)(uintptr_t)(lds_void *)smem;
        __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(A + m0 * lda), 0, (int)(BM * lda * 2), 0x00020000);
        __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(B + n0 * ldb), 0, (int)(BN * ldb * 2), 0x00020000);
        uint32_t voa[2], vob[2];
        {
            const int lane = threadIdx.x & 63, rl = lane / CPR, sl = lane % CPR;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int c = 16 * (sl ^ (((rl >> 1) + 4 * p) & 7));
                voa[p] = (uint32_t)(rl * lda * 2 + c);
                vob[p] = (uint32_t)(rl * ldb * 2 + c);
            }
        }
        issue(s0, ra, rb, lda, ldb, 0, w, voa, vob);
        if (nk > 1) {
            issue(s0 + STAGE, ra, rb, lda, ldb, BK, w, voa, vob);
            wait_vmcnt<AI + BI>();
        } else {
            wait_vmcnt<0>();
        }
        lds_barrier();
        Frag f[2][NF];
        load_frags(smem, 0, f[0]);
        for (int kt = 0; kt < nk - 1; ++kt) {
            const char *cur = smem + (kt & 1) * STAGE;
#pragma unroll
            for (int q = 0; q < NKK - 1; ++q) {
                load_frags(cur, (q + 1) * Mf::KI, f[(q + 1) & 1]);
                mmas(f[q & 1]);
                interleave();
            }
            // stage kt + 1, issued one stage ago, has landed and this wave's last
            // reads of stage kt have returned; then the same for every wave
            wait_vmcnt_lds<0>();
            lds_barrier();
            load_frags(smem + ((kt + 1) & 1) * STAGE, 0, f[0]);
            mmas(f[1]);
            interleave();
            if (kt + 2 < nk) issue(s0 + (kt & 1) * STAGE, ra, rb, lda, ldb, (int64_t)(kt + 2) * BK, w, voa, vob);
        }
        const char *cur = smem + ((nk - 1) & 1) * STAGE;
#pragma unroll
        for (int q = 0; q < NKK - 1; ++q) {
            load_frags(cur, (q + 1) * Mf::KI, f[(q + 1) & 1]);
            mmas(f[q & 1]);
            interleave();
        }
        mmas(f[1]);
        wait_vmcnt_lds<0>();
        lds_barrier();
    }

    __device__ static inline int half() { return 0; }
    __device__ static inline int row_of(int i, int r) {
        const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) % WM;
        return wm * WTM * Mf::M + i * Mf::M + Mf::crow(lane, r);
    }
    __device__ static inline int col_of(int j) {
        const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) / WM;
        return wn * WTN * Mf::M + j * Mf::M + Mf::ccol(lane);
    }
};

// ---------------------------------------------------------------------------
// FP64 and FP32 core fed by direct global->LDS loads, for every contraction of
// those types (distance Gram, score Gram, residual and panel products, FP64 and
// FP32 levels).  One of their MFMAs holds its matrix pipe for 64 cycles, so
// neither LDS nor L2 bandwidth bounds a tile; what costs time is every cycle in
// which all waves of a SIMD wait at once: a register-staged core stored the
// next k-tile and met a barrier after its last MFMA (FP64 matrix pipes 74-84 %
// busy).  Here the fragments of k-group q + 1 are read while the MFMAs of group
// q run, and the barrier lies before the last group's MFMAs, whose fragments
// are already in registers, so the next k-tile's first fragments arrive under
// them.
//
// LDS rows of 128 bytes (16 doubles, 32 floats) with the 16-byte chunks
// XOR-swizzled by (row >> 1) & 7.  A k-tile is four groups of 32 bytes of every
// row; of group q, lane l reads chunk 2 q + (l >> 5) of row l % M: for FP64 the
// half (l >> 4) & 1 of it (one MFMA of 4 k), for FP32 the whole (four MFMAs of
// two k each, k and k + 4 together).  Each phase of such a read covers the 64
// banks once.  NS: LDS stages (2 for the large tiles, whose k-tile takes
// microseconds; 3 or 4 where it is nearer the load latency).  The k order of
// every sum is the same for every tile shape, so the results are the same bits.
// WK = 2 (FP32 levels, small FP64 levels, panel products of one workgroup per
// CU): twice the waves, each half of them taking two of a stage's four groups, so
// that a SIMD has another wave's MFMAs while one waits; these have their own order.
//
// Measured at 256 x 16384 x 16384 in FP64 (the residual product's shape) on one
// card, in bursts: 256 x 128 tiles of 8 waves 1.86 ms (74 TFLOP/s), 128 x 128 of
// 8 waves 1.89, 128 x 64 of 4 waves 1.95, 64 x 64 of 4 waves 2.02; the
// register-staged core 2.08-2.30.  Reading a symmetric B as B^T (k-tiles of 1 KB
// rows), which had paid there, gives nothing here (1.88).
template <typename T> struct RowMf;
template <> struct RowMf<double> : MfmaF64 {
    using Frag = double;
    static constexpr int STEPS = 1;
    __device__ static inline int within(int lane) { return 8 * ((lane >> 4) & 1); }   // byte of the chunk
    __device__ static inline AccV step(const Frag &a, const Frag &b, const AccV &c, int) {
        return MfmaF64::mma(a, b, c);
    }
};
template <> struct RowMf<float> : MfmaF32 {
    using Frag = f32x4;
    static constexpr int STEPS = 4;
    __device__ static inline int within(int) { return 0; }
    __device__ static inline AccV step(const Frag &a, const Frag &b, const AccV &c, int s) {
        return MfmaF32::mma(a[s], b[s], c);
    }
};

// FAR: the operands' rows lie more than 2^32 bytes apart from a tile's first to its
// last, which the buffer loads' 32-bit offsets do not reach: the same loads by
// 64-bit addresses.
template <typename E, int BM, int BN, int WM, int WN, int NS = 2, int WK = 1, bool FAR = false>
struct RowCore {
    using T = E;
    using MF = RowMf<T>;
    using Frag = typename MF::Frag;
    using AccV = typename MF::AccV;
    static constexpr int M = MF::M;
    static constexpr int ROWB = 128;                 // bytes per LDS row
    static constexpr int BK = ROWB / (int)sizeof(T);
    static constexpr int TBM = BM, TBN = BN;
    static constexpr int NW = WM * WN * WK, NT = NW * 64;
    static constexpr int STAGE = (BM + BN) * ROWB;
    static constexpr size_t SMEM = (size_t)NS * STAGE;
    static constexpr int WTM = BM / WM / M, WTN = BN / WN / M;
    // 1 KB loads (8 rows) per wave and stage; where they do not divide evenly
    // the last block is loaded more than once (the same bytes to the same
    // place), so that every wave counts the same number
    static constexpr int AB = BM / 8, BB = BN / 8;
    static constexpr int AI = (AB + NW - 1) / NW, BI = (BB + NW - 1) / NW;
    static constexpr int NKK = 4 / WK;               // k-groups of a stage per wave
    static constexpr int NF = WTM + WTN, NM = WTM * WTN * MF::STEPS;
    static_assert(WTM * WM * M == BM && WTN * WN * M == BN, "whole wave tiles");
    static_assert(WTM >= 1 && WTN >= 1 && NS >= 2 && (WK == 1 || WK == 2), "tile shape");

    AccV acc[WTM][WTN];

    // One operand panel as its loads address it: the resource, and this lane's
    // offset in an even and an odd block of 8 rows (FAR: from its row's start).
    struct Panel {
        __amdgpu_buffer_rsrc_t rsrc;
        const char *row;
        int64_t ld;
        uint32_t v0, v1;
    };
    __device__ static inline Panel panel(const T *A, int64_t ld, int64_t first, int rows) {
        const int rl = (threadIdx.x & 63) >> 3, sl = threadIdx.x & 7;
        const uint32_t o = FAR ? 0 : (uint32_t)(rl * ld * (int)sizeof(T));
        Panel p;
        if (!FAR)
            p.rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(A + first * ld), 0,
                                                       (int)(rows * ld * (int)sizeof(T)), 0x00020000);
        p.row = (const char *)(A + (first + rl) * ld);
        p.ld = ld;
        p.v0 = o + 16 * (sl ^ (rl >> 1));
        p.v1 = o + 16 * (sl ^ ((rl >> 1) + 4));
        return p;
    }
    // Block `blk` of 8 rows of the k-tile starting at element k0 into LDS at `dst`.
    __device__ static inline void load_block(const Panel &p, uint32_t dst, int blk, int64_t k0) {
        const int64_t o = ((int64_t)(blk * 8) * p.ld + k0) * (int)sizeof(T);
        if constexpr (FAR)
            __builtin_amdgcn_global_load_lds((const glb_void *)(p.row + o + (blk & 1 ? p.v1 : p.v0)),
                                             (lds_void *)(uintptr_t)dst, 16, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(p.rsrc, (lds_void *)(uintptr_t)dst, 16,
                                                     blk & 1 ? p.v1 : p.v0, (uint32_t)o, 0, 0);
    }

    // Loads of the k-tile starting at element k0 into the LDS stage at byte
    // offset `stage`.
    __device__ inline void issue(uint32_t stage, const Panel &pa, const Panel &pb, int64_t k0, int w) {
#pragma unroll
        for (int q = 0; q < AI; ++q) {
            int blk = w + q * NW;
            if (AB % NW) blk = blk < AB ? blk : AB - 1;
            load_block(pa, stage + blk * 1024, blk, k0);
        }
#pragma unroll
        for (int q = 0; q < BI; ++q) {
            int blk = w + q * NW;
            if (BB % NW) blk = blk < BB ? blk : BB - 1;
            load_block(pb, stage + BM * ROWB + blk * 1024, blk, k0);
        }
    }

    __device__ inline void load_frags(const char *s, int q, Frag *f) {
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        const int wm = wid % WM, wn = wid / WM % WN;
        const char *sA = s, *sB = s + BM * ROWB;
        const int c = 2 * (NKK * half() + q) + (lane >> 5), in = MF::within(lane);
#pragma unroll
        for (int i = 0; i < WTM; ++i) {
            const int row = (wm * WTM + i) * M + lane % M;
            f[i] = *(const Frag *)(sA + row * ROWB + 16 * (c ^ ((row >> 1) & 7)) + in);
        }
#pragma unroll
        for (int j = 0; j < WTN; ++j) {
            const int row = (wn * WTN + j) * M + lane % M;
            f[WTM + j] = *(const Frag *)(sB + row * ROWB + 16 * (c ^ ((row >> 1) & 7)) + in);
        }
    }

    __device__ inline void mmas(const Frag *f) {
#pragma unroll
        for (int s = 0; s < MF::STEPS; ++s)
#pragma unroll
            for (int i = 0; i < WTM; ++i)
#pragma unroll
                for (int j = 0; j < WTN; ++j) acc[i][j] = MF::step(f[i], f[WTM + j], acc[i][j], s);
    }

    template <int I = 0> __device__ static inline void interleave() {
        constexpr int G = NF > NM ? NF : NM;
        constexpr int nd = (I + 1) * NF / G - I * NF / G;
        constexpr int nm = (I + 1) * NM / G - I * NM / G;
        if constexpr (nd > 0) __builtin_amdgcn_sched_group_barrier(0x100, nd, 0);
        if constexpr (nm > 0) __builtin_amdgcn_sched_group_barrier(0x008, nm, 0);
        if constexpr (I + 1 < G) interleave<I + 1>();
    }

    __device__ inline void negate() {
#pragma unroll
        for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int j = 0; j < WTN; ++j)
#pragma unroll
                for (int r = 0; r < MF::R; ++r) acc[i][j][r] = -acc[i][j][r];
    }

    // Full K loop (K a multiple of BK; rows m0.. and n0.. inside the
    // allocations).  smem holds SMEM bytes and is free again on return.
    // DIFF: the second half of the k range minus the first (the sums are
    // negated half way, which is exact; K a multiple of 2 BK).
    template <bool DIFF = false>
    __device__ inline void run(const T *A, int64_t lda, const T *B, int64_t ldb, int64_t m0,
                               int64_t n0, int64_t K, T *smem_t) {
        char *smem = (char *)smem_t;
#pragma unroll
        for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int j = 0; j < WTN; ++j)
#pragma unroll
                for (int r = 0; r < MF::R; ++r) acc[i][j][r] = 0;
        const int nk = (int)(K / BK);
        if (nk == 0) return;
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t s0 = (uint32_t)(uintptr_t)(lds_void *)smem;
        const Panel pa = panel(A, lda, m0, BM), pb = panel(B, ldb, n0, BN);
        // the first NS stages, then wait for stage 0
#pragma unroll
        for (int p = 0; p < NS; ++p)
            if (p < nk) issue(s0 + p * STAGE, pa, pb, (int64_t)p * BK, w);
        if (nk >= NS) wait_vmcnt<(NS - 1) * (AI + BI)>();
        else wait_vmcnt<0>();
        lds_barrier();
        Frag f[2][NF];
        load_frags(smem, 0, f[0]);
        int cur = 0;
        for (int kt = 0; kt < nk - 1; ++kt) {
            const char *sc = smem + cur * STAGE;
            const int nxt = cur + 1 == NS ? 0 : cur + 1;
            if (DIFF && 2 * kt == nk) negate();
#pragma unroll
            for (int q = 0; q < NKK - 1; ++q) {
                load_frags(sc, q + 1, f[(q + 1) & 1]);
                mmas(f[q & 1]);
                interleave();
            }
            // stage kt + 1 has landed (up to NS - 2 later stages may be in
            // flight; near the end fewer are, so wait for all) and this wave's
            // last reads of stage kt have returned; then the same for every wave
            if (kt + NS - 1 < nk) wait_vmcnt_lds<(NS - 2) * (AI + BI)>();
            else wait_vmcnt_lds<0>();
            lds_barrier();
            load_frags(smem + nxt * STAGE, 0, f[0]);
            mmas(f[1]);
            interleave();
            // nobody reads stage kt any more
            if (kt + NS < nk) issue(s0 + cur * STAGE, pa, pb, (int64_t)(kt + NS) * BK, w);
            cur = nxt;
        }
        const char *sc = smem + cur * STAGE;
        if (DIFF && nk == 2) negate();
#pragma unroll
        for (int q = 0; q < NKK - 1; ++q) {
            load_frags(sc, q + 1, f[(q + 1) & 1]);
            mmas(f[q & 1]);
            interleave();
        }
        mmas(f[1]);
        wait_vmcnt_lds<0>();
        lds_barrier();
        if constexpr (WK == 2) {
            static_assert(WTM * WTN * MF::R * WM * WN * 64 * sizeof(T) <= SMEM, "the other half's sums");
            T *const other = (T *)smem + threadIdx.x % (WM * WN * 64);
            if (half()) {
#pragma unroll
                for (int i = 0; i < WTM; ++i)
#pragma unroll
                    for (int j = 0; j < WTN; ++j)
#pragma unroll
                        for (int r = 0; r < MF::R; ++r)
                            other[((i * WTN + j) * MF::R + r) * (WM * WN * 64)] = acc[i][j][r];
            }
            __syncthreads();
            if (!half()) {
#pragma unroll
                for (int i = 0; i < WTM; ++i)
#pragma unroll
                    for (int j = 0; j < WTN; ++j)
#pragma unroll
                        for (int r = 0; r < MF::R; ++r)
                            acc[i][j][r] += other[((i * WTN + j) * MF::R + r) * (WM * WN * 64)];
            }
        }
    }

    // WK = 2: which half of every stage's k-groups this wave sums; the sums are
    // those of the waves of half 0 after run().
    __device__ static inline int half() { return WK == 1 ? 0 : (int)(threadIdx.x >> 6) / (WM * WN); }
    __device__ static inline int row_of(int i, int r) {
        const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) % WM;
        return (wm * WTM + i) * M + MF::crow(lane, r);
    }
    __device__ static inline int col_of(int j) {
        const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) / WM % WN;
        return (wn * WTN + j) * M + MF::ccol(lane);
    }
};

template <int BM, int BN, int WM, int WN, int NS = 2, bool FAR = false>
using Dma64Core = RowCore<double, BM, BN, WM, WN, NS, 1, FAR>;

} // namespace cdl
