// bf16 GEMM  out = epilogue(A W^T + bias)  for gfx950, fp32 accumulation on the matrix cores.
//
// This is the "24 b L_q C^2" term of the per-layer cost in Appendix B of the paper (QKV, output
// and FFN projections), plus the cross-attention projections the cost model leaves out.
//
// Two kernels on the matrix cores.  gemm_alt64_kernel (16x16x32 MFMAs, direct global -> LDS loads, persistent) serves
// every shape whose operands (16-byte aligned), and 128 rows of the output, are below 4 GiB: it uses 32-bit byte offsets
// per lane.  gemm_kernel (32x32x16 MFMAs, tiles staged through registers, 64-bit addresses) serves the others.  Both
// operands are K-contiguous (activations [M, K], weights [N, K]), so fragments are plain 16-byte pieces of rows.
//   Split-K (few output tiles, long k: FFN-2 of one chunk) is two launches: the parts store fp32 partial sums, a second
// kernel adds them in k order and applies the epilogue, and the LayerNorm that follows if there is one.  fp32 atomics
// on the output cost ~40 us per 1.5 M elements here, and a last-arriver reduction inside one launch needs device-scope
// fences that write back and invalidate the whole L2 of an XCD (measured +100 us on a 64 us launch).
#include "common.h"

#include <mutex>
#include <type_traits>
#include <utility>

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

namespace sdv2 {

namespace {

// Epilogue.  Accumulator register r of a 32x32 block holds row 8 (r / 4) + 4 (lane / 32) + r % 4 and
// column lane % 32, which is a poor shape for memory (2-byte or 4-byte pieces of many rows).  Each wave
// therefore passes its accumulators through a private LDS region, 32 rows x 64 columns at a time, and
// reads them back row-major so that a lane owns four consecutive columns: stores become 8-byte (bf16)
// or 16-byte (fp32) pieces that fill whole 128- or 256-byte row segments, and the read-modify-write
// epilogues issue all their loads of x before the first use.
constexpr int EPI_LD = 68;                          // floats per LDS row: 64 + 4 of padding
constexpr int EPI_WAVE_FLOATS = 32 * EPI_LD;

template <int EPI, int NB>
__device__ __forceinline__ void epilogue_chunk(const GemmArgs& g, const f32x16& acc0, const f32x16& acc1, float* stage,
                                               int row_base, int col_base, int lane) {
    const int l31 = lane & 31, lh = lane >> 5;
    __builtin_amdgcn_sched_barrier(0);               // one chunk at a time: bounds the registers in flight
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * lh + (r & 3);
        stage[row * EPI_LD + l31] = acc0[r];
        if (NB == 2) stage[row * EPI_LD + 32 + l31] = acc1[r];
    }
    constexpr int kLanesPerRow = NB * 8;
    constexpr int kRowsPerPass = 64 / kLanesPerRow;
    constexpr int kPasses = 32 / kRowsPerPass;
    const int prow = lane / kLanesPerRow;
    const int c4 = (lane % kLanesPerRow) * 4;
    const int gcol = col_base + c4;
    const bool col_ok = gcol < g.N;                  // N is a multiple of 4: all four columns or none
    const int gcolc = col_ok ? gcol : 0;
    f32x4 bias = {0.0f, 0.0f, 0.0f, 0.0f};
    if (g.bias != nullptr) bias = *reinterpret_cast<const f32x4*>(g.bias + gcolc);
    f32x4 gate_a = {0.0f, 0.0f, 0.0f, 0.0f};
    if (EPI == kEpiGatedResidual) gate_a = *reinterpret_cast<const f32x4*>(g.gate_a + gcolc);
    // passes are handled four at a time: all loads of x and of the gate first, then the arithmetic and stores
    constexpr int kGroup = kPasses < 4 ? kPasses : 4;
#pragma unroll
    for (int p0 = 0; p0 < kPasses; p0 += kGroup) {
        f32x4 xv[kGroup];
        f32x4 gb[kGroup];
        if (EPI == kEpiGatedResidual || EPI == kEpiResidual) {
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                const int grow = row_base + (p0 + q) * kRowsPerPass + prow;
                const bool ok = col_ok && grow < g.M;
                const int growc = ok ? grow : 0;
                xv[q] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.out) + (size_t)growc * g.N + gcolc);
                if (EPI == kEpiGatedResidual)
                    gb[q] = *reinterpret_cast<const f32x4*>(g.gate_b + (size_t)(growc / g.rows_per_gate) * g.gate_b_stride + gcolc);
            }
        }
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            const int row = (p0 + q) * kRowsPerPass + prow;
            const int grow = row_base + row;
            f32x4 v = *reinterpret_cast<const f32x4*>(stage + row * EPI_LD + c4);
            v += bias;
            if (col_ok && grow < g.M) {
                const size_t o = (size_t)grow * g.N + gcol;
                if (EPI == kEpiPartial) {
                    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.out) + o) = v;
                } else if (EPI == kEpiBias || EPI == kEpiBiasGelu) {
                    bf16x4 w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = (bf16)(EPI == kEpiBiasGelu ? gelu_tanh_f(v[e]) : v[e]);
                    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(g.out) + o) = w;
                } else {
                    if (EPI == kEpiGatedResidual) v *= (gate_a + gb[q]);
                    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.out) + o) = xv[q] + v;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// row0: first output row of this wave's tile; col0: first output column of the workgroup's tile.
template <int TM, int TN, int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs& g, f32x16 (&acc)[TM][TN], float* stage, int row0, int col0,
                                         int lane) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int jc = 0; jc < (TN + 1) / 2; ++jc) {
            if (2 * jc + 1 < TN)
                epilogue_chunk<EPI, 2>(g, acc[i][2 * jc], acc[i][2 * jc + 1], stage, row0 + 32 * i, col0 + 64 * jc, lane);
            else
                epilogue_chunk<EPI, 1>(g, acc[i][2 * jc], acc[i][2 * jc], stage, row0 + 32 * i, col0 + 64 * jc, lane);
        }
    }
}

template <int TM, int TN>
__device__ __forceinline__ void run_epilogue(const GemmArgs& g, f32x16 (&acc)[TM][TN], float* stage, int row0, int col0,
                                             int lane) {
    switch (g.epilogue) {
        case kEpiBias: epilogue<TM, TN, kEpiBias>(g, acc, stage, row0, col0, lane); break;
        case kEpiBiasGelu: epilogue<TM, TN, kEpiBiasGelu>(g, acc, stage, row0, col0, lane); break;
        case kEpiGatedResidual: epilogue<TM, TN, kEpiGatedResidual>(g, acc, stage, row0, col0, lane); break;
        case kEpiPartial: epilogue<TM, TN, kEpiPartial>(g, acc, stage, row0, col0, lane); break;
        default: epilogue<TM, TN, kEpiResidual>(g, acc, stage, row0, col0, lane); break;
    }
}

// The register-staged kernel: workgroup of four waves stacked along M, wave tile (32 TM) x (32 TN), workgroup tile
// (128 TM) x (32 TN) x 64; global -> registers -> LDS (two LDS stages), one barrier per k tile.
// Tiles whose k loop fits in 256 registers are compiled for two workgroups per compute unit, so that one
// workgroup's barrier and LDS-latency bubbles are filled by the other's MFMAs.  BK (64 or 128) is the k
// depth of an LDS stage: a deeper stage halves the number of barriers, which is what the small tiles
// (few MFMAs per barrier) are short of.
// PF is the number of register sets = how many k tiles ahead the global loads run.  A compute unit needs
// on the order of 100 KB of loads in flight to cover the L2 latency; tiles that run one workgroup per
// unit get there with three sets, small tiles with two sets and two or three workgroups per unit.
template <int TM, int TN, int BK, int PF>
__global__ __launch_bounds__(256, ((TM * TN <= 5 && BK == 64 && PF == 2) ? 2 : 1)) void gemm_kernel(GemmArgs g, int tiles_m,
                                                                                                  int tiles_n, int group_m,
                                                                                                  int splitk) {
    constexpr int BM = 128 * TM;
    constexpr int BN = 32 * TN;
    constexpr int CPR = BK / 8;                 // 16-byte chunks per LDS row
    constexpr int RPP = 256 / CPR;              // tile rows covered by one pass of the 256 threads
    constexpr int NA = BM / RPP;                // 16-byte chunks of the A tile per thread
    constexpr int NB = BN / RPP;                // of the W tile
    constexpr int KS = BK / 16;                 // MFMA k steps per stage
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16* const sm = reinterpret_cast<bf16*>(smem_raw);     // [2][BM*BK | BN*BK]
    constexpr int STAGE = (BM + BN) * BK;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int l31 = lane & 31;
    const int lh = lane >> 5;

    // ---- which tile: undo the round-robin XCD dispatch, then grouped ordering
    const int nwg = gridDim.x;                                   // multiple of 8
    const int logical = (blockIdx.x & 7) * (nwg >> 3) + (blockIdx.x >> 3);
    const int tiles = tiles_m * tiles_n;
    if (logical >= tiles * splitk) return;
    const int ks = logical / tiles;                              // which part of k (0 when k is not split)
    const int t = logical - ks * tiles;
    const int group_size = group_m * tiles_n;
    const int grp = t / group_size;
    const int first_m = grp * group_m;
    const int gm = min(tiles_m - first_m, group_m);
    const int in_grp = t - grp * group_size;
    const int tile_m = first_m + in_grp % gm;
    const int tile_n = in_grp / gm;
    const int m0 = tile_m * BM;
    const int n0 = tile_n * BN;

    const int KT = g.K / BK;
    const int kt0 = (int)((long long)ks * KT / splitk);
    const int kt1 = (int)((long long)(ks + 1) * KT / splitk);
    if (splitk > 1) {                                            // this part's fp32 partial sums, plain stores
        g.out = g.splitk_partials + (size_t)ks * g.M * g.N;
        g.epilogue = kEpiPartial;
        g.bias = nullptr;
    }

    // ---- global -> register staging
    const int crow = tid / CPR;
    const int cchunk = tid % CPR;
    const bf16* ap[NA];
    const bf16* bp[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = min(m0 + crow + RPP * i, g.M - 1);
        ap[i] = g.a + (size_t)row * g.K + cchunk * 8;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = min(n0 + crow + RPP * i, g.N - 1);
        bp[i] = g.w + (size_t)row * g.K + cchunk * 8;
    }
    // LDS swizzle: the 16-byte chunk c of row r is stored at position c ^ ((r / 2) % 8).  The LDS has 64
    // banks (256 bytes per clock); a row is 128 bytes, so rows r and r + 1 fall in different bank halves
    // and the sixteen lanes that a b128 read serves per clock (rows r .. r + 15, same chunk) then hit
    // sixteen different 16-byte slots.  (XOR with r % 8, the 32-bank recipe, reads at half rate here.)
    // RPP is a multiple of 16, so ((row / 2) % 8) of every chunk this thread stages is that of crow.
    const int st_off = crow * BK + ((cchunk ^ ((crow >> 1) & 7)) << 3);
    // PF register sets: tile t lives in set t % PF from its load until it is written to LDS stage t % 2
    // at the end of iteration t - 1, so a global load has PF iterations of MFMA work to hide behind.
    bf16x8 ra[PF][NA], rb[PF][NB];

    auto gload = [&](bf16x8 (&xa)[NA], bf16x8 (&xb)[NB], int kt) {
#pragma unroll
        for (int i = 0; i < NA; ++i) xa[i] = *reinterpret_cast<const bf16x8*>(ap[i] + kt * BK);
#pragma unroll
        for (int i = 0; i < NB; ++i) xb[i] = *reinterpret_cast<const bf16x8*>(bp[i] + kt * BK);
    };
    auto sstore = [&](const bf16x8 (&xa)[NA], const bf16x8 (&xb)[NB], int buf) {
        bf16* sa = sm + buf * STAGE;
        bf16* sb = sa + BM * BK;
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<bf16x8*>(sa + st_off + i * RPP * BK) = xa[i];
#pragma unroll
        for (int i = 0; i < NB; ++i) *reinterpret_cast<bf16x8*>(sb + st_off + i * RPP * BK) = xb[i];
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int a_row0 = wave * (32 * TM) + l31;
    // One stage = KS 16-wide steps.  The fragments of step s + 1 are read from LDS before the MFMAs of
    // step s are issued, so that the LDS latency hides behind matrix work.
    auto load_frags = [&](bf16x8 (&fa)[TM], bf16x8 (&fb)[TN], const bf16* sa, const bf16* sb, int s) {
        const int coff = ((2 * s + lh) ^ ((l31 >> 1) & 7)) << 3;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[i] = *reinterpret_cast<const bf16x8*>(sa + (a_row0 + 32 * i) * BK + coff);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            fb[j] = *reinterpret_cast<const bf16x8*>(sb + (l31 + 32 * j) * BK + coff);
    };
    auto compute = [&](int buf) {
        const bf16* sa = sm + buf * STAGE;
        const bf16* sb = sa + BM * BK;
        bf16x8 fa[2][TM], fb[2][TN];
        load_frags(fa[0], fb[0], sa, sb, 0);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s + 1 < KS) load_frags(fa[(s + 1) & 1], fb[(s + 1) & 1], sa, sb, s + 1);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s & 1][i], fb[s & 1][j], acc[i][j], 0, 0, 0);
        }
    };

    // Issue order of one half iteration.  A wave issues in order, and a global load or an LDS write
    // occupies its issue slot for tens of cycles; so they are spread between the MFMAs (whose 32-cycle
    // execution leaves issue slots free) instead of being issued in a burst before or after them:
    //   first step's fragment reads | per MFMA: 1 MFMA, fragment reads of the next step, then one
    //   global load (tile i + 2) in the first half of the MFMAs and one LDS write (tile i + 1) in the
    //   second half.
    auto issue_pipeline = [&]() {
        constexpr int kMfma = TM * TN * KS;
        constexpr int kReadsPerMfma = (TM + TN + TM * TN - 1) / (TM * TN);
        constexpr int kMem = NA + NB;
        constexpr int kMemPerMfma = (2 * kMem + kMfma - 1) / kMfma;
        __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);
#pragma unroll
        for (int m = 0; m < kMfma; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, kReadsPerMfma, 0);
            if (m < kMfma / 2) __builtin_amdgcn_sched_group_barrier(0x020, kMemPerMfma, 0);
            else __builtin_amdgcn_sched_group_barrier(0x200, kMemPerMfma, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // Loads are unconditional (the tile index is clamped, the tail re-reads the last tile) so that a step
    // has no control flow around them and they stay in flight across the MFMA work.  Step k of the
    // unrolled body: tile t sits in LDS stage k % 2; load tile t + PF into set k % PF (free since tile t
    // was written out), compute, write set (k + 1) % PF (tile t + 1) to the other stage.
    const int nk = kt1 - kt0;
    const int kt_last = kt1 - 1;
    auto step = [&](auto kc, int t) {
        constexpr int k = decltype(kc)::value;
        __builtin_amdgcn_sched_barrier(0);
        gload(ra[k % PF], rb[k % PF], min(kt0 + t + PF, kt_last));
        compute(k % 2);
        sstore(ra[(k + 1) % PF], rb[(k + 1) % PF], (k + 1) % 2);
        issue_pipeline();
        __syncthreads();
    };
    if (nk > 0) {
#pragma unroll
        for (int p = 0; p < PF; ++p) gload(ra[p], rb[p], min(kt0 + p, kt_last));
        sstore(ra[0], rb[0], 0);
    }
    __syncthreads();
    constexpr int U = (PF % 2 == 0) ? PF : 2 * PF;      // unroll so that stage and set indices are constants
    int i = 0;
    for (; i + U <= nk; i += U) {
        step(std::integral_constant<int, 0>{}, i);
        step(std::integral_constant<int, 1>{}, i + 1);
        if constexpr (U > 2) {
            step(std::integral_constant<int, 2>{}, i + 2);
            step(std::integral_constant<int, 3>{}, i + 3);
            step(std::integral_constant<int, 4>{}, i + 4);
            step(std::integral_constant<int, 5>{}, i + 5);
        }
    }
    // tail: fewer than U tiles left; the last tile needs no write-out but doing one is harmless
    if (i < nk) step(std::integral_constant<int, 0>{}, i);
    if constexpr (U > 2) {
        if (i + 1 < nk) step(std::integral_constant<int, 1>{}, i + 1);
        if (i + 2 < nk) step(std::integral_constant<int, 2>{}, i + 2);
        if (i + 3 < nk) step(std::integral_constant<int, 3>{}, i + 3);
        if (i + 4 < nk) step(std::integral_constant<int, 4>{}, i + 4);
    }

    // ---- epilogue (the LDS stages are free once every wave has left the k loop)
    __syncthreads();
    float* stage = reinterpret_cast<float*>(smem_raw) + wave * EPI_WAVE_FLOATS;
    run_epilogue<TM, TN>(g, acc, stage, m0 + wave * (32 * TM), n0, lane);
}

// ---------------------------------------------------------------------------------------------------
// Second kernel, for every shape within 32-bit byte offsets (fits_32bit_offsets): v_mfma_f32_16x16x32_bf16 on tiles that go
// global -> LDS directly (global_load_lds_dwordx4: no staging registers, no LDS write instructions).
//
//   What bounds it.  On random data the chip is power limited: a register-resident loop of 32x32x16 MFMAs sustains
// 1.82 PFLOP/s, of 16x16x32 MFMAs 2.05 PFLOP/s (2.48 / 2.45 on zeros), because the smaller instruction moves half of
// the accumulator data per flop.  Below that it is the LDS pipeline: 4.6 clocks per fragment read of 1 KB and 16 to 25
// per direct load of 1 KB, against 16 clocks per MFMA.  Hence large wave tiles (128 x 64 of a 256 x 256 workgroup
// tile: 24 fragment reads per 64 MFMAs of a k tile of 64), whole 128-byte lines per load, and tiles as large as the
// shape allows (a 1024-row product streams its operands through the L2s at up to 19 TB/s: 128 x 160 tiles on 256
// units, 62 us for 1024 x 5120 x 5120 where 128 x 160 register-staged tiles took 67).
//   Main loop.  A k tile is 64 wide and holds two MFMA k steps ("halves") that take turns, whence the name.  While the
// MFMAs of one half are issued, the fragments of the other half are read from LDS, and (second half) the tile loads go out,
// one every few MFMAs:
//     half 0 of tile t | wait: tile t + 1 has landed, every fragment of tile t is in registers | barrier |
//     half 1 of tile t, fragments of half 0 of tile t + 1, loads of tile t + stages into the stage tile t has left
// One barrier per k tile, no fragment latency behind it.  The order inside a half is the program order, held by
// scheduling barriers: left to the scheduler the loads of a half are issued in one burst.
//   Stages.  A and W have rings of their own (NSA, NSW stages): weights come from HBM (every layer has its own),
// activations mostly from the L2, so where 160 KB allow it W gets the additional stage.
//   ROLES: half of the waves fetch A, the other half W, each with its own wait count.  With every wave fetching both, a
// wave waits for its loads in issue order and so for the slower operand; with large tiles of few loads per MFMA the
// wait is hidden and sharing the loads evenly is 3 to 8 % faster (256-row tiles), with 128-row tiles roles are
// (1024 x 5120 x 5120: 65 -> 60 us).
//   Persistent: a workgroup takes its tiles in turn, and the loads run on across them: the first k tiles of the next
// output tile are in flight while this one's epilogue stores (1.3B FFN-1 on 8192 rows: 207 -> 188 us).
//   Epilogue from registers: the operands are swapped (W rows are the MFMA's rows), so a lane holds four consecutive
// columns of one row; two bf16 blocks are interleaved with v_permlane16_swap into 16-byte stores, fp32 pieces are 16
// bytes as they are.  No LDS round trip, so the ring can keep filling.
//   The bias joins the finished sum (see store_tile); it is the wave's own 64 to 128 columns, the same for sixteen lanes.
//   XCD-aware order: an XCD (one L2) owns a contiguous range of tiles, ordered in groups of GROUP_M tile rows that share
// weight tiles.
//   Tried and dropped: W fragments straight from global memory into registers, A through LDS (16 rows of 64 bytes per
// load: 20 to 40 % slower on every shape); 256 x 256 with four waves of 128 x 128 (a third fewer fragment reads, but one
// wave per SIMD leaves the barrier and the epilogue uncovered: equal on square shapes, 15 % slower at k = 1536); NSW = 5 with NSA = 3 on 128 x 160 (same as 4 and 4).
constexpr int vmcnt_only(int n) {     // s_waitcnt with only vmcnt constrained
    return (n & 0xF) | ((n >> 4) << 14) | 0x0F70;
}
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(4))) float* scalar_float_ptr;      // read through the scalar cache where uniform
typedef __attribute__((address_space(3))) unsigned char* lds_byte_ptr;     // 32 bits; a generic pointer is tested for null at every cast
// 16 bytes per lane from a buffer straight into LDS at dst + 16 * lane (dst is wave-uniform): byte offsets of the lane and of
// the wave, 32 bits each.
__device__ __forceinline__ void load_to_lds_b128(__amdgpu_buffer_rsrc_t src, uint32_t lane_off, uint32_t wave_off, lds_byte_ptr dst) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void_ptr)dst, 16, (int)lane_off, (int)wave_off, 0, 0);
}
// The same from a 64-bit address.
__device__ __forceinline__ void load_to_lds_b128(const unsigned char* src, lds_byte_ptr dst) {
    __builtin_amdgcn_global_load_lds(src, (lds_void_ptr)dst, 16, 0, 0);
}
// A buffer of plain bytes (word 3: 32-bit data, no swizzle), below 4 GiB.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t byte_buffer(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl(std::make_integer_sequence<int, N>{}, f); }

// Stores a wave's tile.  acc[i][j][r] is the element (16 i + lane % 16, 16 j + 4 (lane / 16) + r) of it.  FULL: the tile
// lies inside the output.  bias_own: the bias of column block lane % 16; SCALAR: it is fetched here instead, through the
// scalar cache (the wave's columns are uniform).  The bias joins the finished sum: an accumulator
// that starts from it rounds every partial sum at the bias's magnitude (1024 x 1536 x 1536, relative error against 64 bits:
// 1.4e-7 after, 3.1e-7 from a bias of the result's size, 2.6e-8 and 3.5e-7 from one 40 times as large).  xpre: x read at the
// start of the tile (small tiles), else x is read here, a block of rows ahead of its use.
template <int TM, int TN, int EPI, bool FULL, bool SCALAR>
__device__ __forceinline__ void store_tile(const GemmArgs& g, void* outp, f32x4 (&acc)[TM][TN], const f32x4& bias_own, int row0, int col0, int lane,
                                           const f32x4* xpre = nullptr) {
    const int l15 = lane & 15, lq = lane >> 4;
    const int rows = FULL ? 16 * TM : min(16 * TM, g.M - row0);
    static_assert(TN <= 16, "a row of lanes holds the bias of its column blocks");
    f32x4 bias[TN];
    if constexpr (!SCALAR) {
        static_for<TN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[j][e] = dpp_f<0x150 + j>(bias_own[e]);      // row_newbcast: lane j of the row of 16
        });
    } else {
        const bool any = g.bias != nullptr;
        const scalar_float_ptr s = (scalar_float_ptr)reinterpret_cast<uintptr_t>(g.bias);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            bias[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (any) {
                const int c = col0 + 16 * j < g.N ? col0 + 16 * j : 0;                        // N is a multiple of 16
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float b0 = s[c + e], b1 = s[c + 4 + e], b2 = s[c + 8 + e], b3 = s[c + 12 + e];
                    asm("" : "+s"(b0), "+s"(b1), "+s"(b2), "+s"(b3));                           // values to choose from, not addresses
                    bias[j][e] = lq < 2 ? (lq == 0 ? b0 : b1) : (lq == 2 ? b2 : b3);
                }
            }
        }
    }
    if constexpr (EPI == kEpiBias || EPI == kEpiBiasGelu || EPI == kEpiGainSquares) {
        f32x4 gain[EPI == kEpiGainSquares ? TN : 1];
        if constexpr (EPI == kEpiGainSquares) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int c = col0 + 16 * j + 4 * lq;
                gain[j] = *reinterpret_cast<const f32x4*>(g.gain + (FULL || c < g.N ? c : 0));
            }
        }
        unsigned char* const base = reinterpret_cast<unsigned char*>(reinterpret_cast<bf16*>(outp) + (size_t)row0 * g.N);
        auto pack = [&](const f32x4& v, uint32_t& d0, uint32_t& d1) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (bf16)(EPI == kEpiBiasGelu ? gelu_tanh_f(v[e]) : v[e]);
            const uint2 u = __builtin_bit_cast(uint2, w);
            d0 = u.x; d1 = u.y;
        };
        const int cl = col0 + 16 * (lq & 1) + 8 * (lq >> 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            const int r = 16 * i + l15;
            const uint32_t ro = (uint32_t)r * (uint32_t)g.N * 2u;
            f32x4 v[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) v[j] = acc[i][j] + bias[j];
            if constexpr (EPI == kEpiGainSquares) {
                // A lane has 4 TN numbers of a row, the four quarters of the wave together 16 TN of them: one sum per row and wave.
                // In one pass with the stores: a pass of its own, which leaves its sums in acc, cost all epilogues of the kernel
                // up to 40 registers and the 256 x 256 tile 75 spilled ones, whose reloads wait for every tile load in flight.
                float q = 0.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if (FULL || col0 + 16 * j < g.N) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) q += v[j][e] * v[j][e];
                    }
                    v[j] *= gain[j];
                }
                const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(q), __float_as_uint(q), false, false);
                q = __uint_as_float(h[0]) + __uint_as_float(h[1]);
                const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(q), __float_as_uint(q), false, false);
                q = __uint_as_float(p[0]) + __uint_as_float(p[1]);
                if (lq == 0 && r < rows) g.squares[(size_t)(unsigned)(col0 / (16 * TN)) * (unsigned)g.M + (unsigned)(row0 + r)] = q;
            }
#pragma unroll
            for (int j = 0; j + 1 < TN; j += 2) {
                uint32_t a0, a1, b0, b1;
                pack(v[j], a0, a1);
                pack(v[j + 1], b0, b1);
                const auto r0 = __builtin_amdgcn_permlane16_swap(a0, b0, false, false);
                const auto r1 = __builtin_amdgcn_permlane16_swap(a1, b1, false, false);
                uint4 u; u.x = r0[0]; u.y = r1[0]; u.z = r0[1]; u.w = r1[1];
                if (FULL || (r < rows && cl + 16 * j < g.N)) *reinterpret_cast<uint4*>(base + (ro + (uint32_t)(cl + 16 * j) * 2u)) = u;
            }
            if constexpr (TN % 2) {
                uint32_t a0, a1;
                pack(v[TN - 1], a0, a1);
                const int gcol = col0 + 16 * (TN - 1) + 4 * lq;
                uint2 u; u.x = a0; u.y = a1;
                if (FULL || (r < rows && gcol < g.N)) *reinterpret_cast<uint2*>(base + (ro + (uint32_t)gcol * 2u)) = u;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    } else {
        unsigned char* const base = reinterpret_cast<unsigned char*>(reinterpret_cast<float*>(outp) + (size_t)row0 * g.N);
        const bool one_gate = EPI == kEpiGatedResidual && row0 / g.rows_per_gate == (row0 + rows - 1) / g.rows_per_gate;
        constexpr int G = TN % 4 == 0 ? 4 : TN % 3 == 0 ? 3 : TN % 5 == 0 ? 5 : TN % 2 == 0 ? 2 : 1;    // column blocks at a time
#pragma unroll
        for (int j0 = 0; j0 < TN; j0 += G) {
            __builtin_amdgcn_sched_barrier(0);
            const int gcol = col0 + 16 * j0 + 4 * lq;
            f32x4 gate[G];
            auto load_gate = [&](int row) {
                const float* gb = g.gate_b + (size_t)(row / g.rows_per_gate) * g.gate_b_stride;
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    const int c = FULL || gcol + 16 * j < g.N ? gcol + 16 * j : 0;
                    gate[j] = *reinterpret_cast<const f32x4*>(g.gate_a + c) + *reinterpret_cast<const f32x4*>(gb + c);
                }
            };
            if (EPI == kEpiGatedResidual && one_gate) load_gate(row0);
            constexpr int XD = TM * TN > 16 ? 2 : 4;                                // row blocks of x in flight
            f32x4 xv[XD][G];
            auto load_x = [&](int i) {
                const uint32_t ro = (uint32_t)(FULL ? 16 * i + l15 : min(16 * i + l15, rows - 1)) * (uint32_t)g.N * 4u;
#pragma unroll
                for (int j = 0; j < G; ++j)
                    xv[i % XD][j] = *reinterpret_cast<const f32x4*>(base + (ro + (uint32_t)(FULL || gcol + 16 * j < g.N ? gcol + 16 * j : 0) * 4u));
            };
            constexpr bool pre = TM * TN <= 16;
            if (EPI != kEpiPartial && !pre) {
#pragma unroll
                for (int i = 0; i < XD - 1 && i < TM; ++i) load_x(i);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (EPI != kEpiPartial && !pre && i + XD - 1 < TM) load_x(i + XD - 1);
                __builtin_amdgcn_sched_barrier(0);
                const int r = 16 * i + l15;
                if (EPI == kEpiGatedResidual && !one_gate) load_gate(row0 + min(r, rows - 1));
                const uint32_t ro = (uint32_t)r * (uint32_t)g.N * 4u;
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    f32x4 v = acc[i][j0 + j] + bias[j0 + j];
                    if (EPI == kEpiGatedResidual) v *= gate[j];
                    if (EPI != kEpiPartial) v += pre ? xpre[i * TN + j0 + j] : xv[i % XD][j];
                    if (FULL || (r < rows && gcol + 16 * j < g.N)) *reinterpret_cast<f32x4*>(base + (ro + (uint32_t)(gcol + 16 * j) * 4u)) = v;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

template <int TM, int TN, int EPI, bool SCALAR>
__device__ __forceinline__ void store_wave(const GemmArgs& g, void* outp, f32x4 (&acc)[TM][TN], const f32x4& bias_own, int row0, int col0, int lane,
                                           const f32x4* xpre = nullptr) {
    asm volatile("" : "+v"(lane));        // formed anew for every tile: lane terms kept across the k loop would cost it registers
    if (row0 + 16 * TM <= g.M && col0 + 16 * TN <= g.N) store_tile<TM, TN, EPI, true, SCALAR>(g, outp, acc, bias_own, row0, col0, lane, xpre);
    else if (row0 < g.M) store_tile<TM, TN, EPI, false, SCALAR>(g, outp, acc, bias_own, row0, col0, lane, xpre);
}

template <int WM, int WN, int TM, int TN, int NSA, int NSW, bool ROLES, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) void gemm_alt64_kernel(GemmArgs g, int tiles_m, int tiles_n, int group_m, int splitk) {
    const unsigned workgroups = gridDim.x;
#include "gemm_alt64_body.inc"
}

// With workgroups behind its own that fetch memory.  A kernel of its own: in the same one the few instructions more cost every
// launch 1 to 4 %.
template <int WM, int WN, int TM, int TN, int NSA, int NSW, bool ROLES, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) void gemm_fetching_kernel(GemmArgs g, int tiles_m, int tiles_n, int group_m, int splitk,
                                                                          unsigned workgroups, WarmArgs warm) {
    if (blockIdx.x >= workgroups) return warm_memory(warm, blockIdx.x - workgroups);
#include "gemm_alt64_body.inc"
}

struct TilePlan {
    int tm, tn, pf;       // register-staged kernel: tile (128 tm) x (32 tn), pf register sets
    int dma = 0;          // otherwise: a configuration of gemm_alt64_kernel (tm, tn, pf unused)
    int splitk = 1;       // parts of the k range, each its own workgroup (needs scratch)
};

// gemm_alt64_kernel addresses an operand, and the output from the first row of a wave's tile (at most 128 rows of fp32), with
// 32-bit byte offsets per lane: it serves operands below 4 GiB and rows of which that many are below 4 GiB.
bool fits_32bit_offsets(int M, int N, int K) {
    constexpr unsigned long long kLimit = 0xFFFFFFFFull;
    return (unsigned long long)M * K * 2 <= kLimit && (unsigned long long)N * K * 2 <= kLimit &&
           (unsigned long long)(M < 128 ? M : 128) * N * 4 <= kLimit;
}

// Its loads go from global memory to LDS in pieces of 16 bytes, which have to start at multiples of 16; the register-staged
// kernel's are ordinary vector loads, good for any address of a bf16.
bool operands_aligned(const GemmArgs& g) {
    return ((reinterpret_cast<uintptr_t>(g.a) | reinterpret_cast<uintptr_t>(g.w) | reinterpret_cast<uintptr_t>(g.w2)) & 15) == 0;
}

// What it does not serve: the time of the busiest compute unit for the register-staged kernel; one k tile of a
// workgroup costs a fixed part (~0.25 us alone, half of it when a second workgroup fills the bubbles) plus ~21 ns per
// MFMA a wave issues (fitted to a sweep); small tiles fit two workgroups per unit.
TilePlan plan_register_staged(int M, int N, int K) {
    TilePlan best{1, 4, 2};
    double best_cost = 1e300;
    for (int tm = 1; tm <= 2; ++tm) {
        for (int tn = 2; tn <= 7; ++tn) {
            const int wgs = ((M + 128 * tm - 1) / (128 * tm)) * ((N + 32 * tn - 1) / (32 * tn));
            const int occ = (tm * tn <= 5) ? 2 : 1;
            const int per_cu = (wgs + kUnits - 1) / kUnits;
            const double mfma = 0.021 * 4 * tm * tn;
            double cost;
            if (occ == 2 && per_cu >= 2) cost = (per_cu + 1) / 2 * (0.25 + 2 * mfma);
            else cost = per_cu * (0.25 + mfma);
            cost = cost * (K / 64) + per_cu * 0.04 * tm * tn;      // + epilogue
            if (cost < best_cost) {
                best_cost = cost;
                best = TilePlan{tm, tn, 2};
            }
        }
    }
    return best;
}

template <int TM, int TN, int PF>
hipError_t launch_one(const GemmArgs& g, int splitk, hipStream_t s) {
    constexpr int BK = 64;
    constexpr int BM = 128 * TM, BN = 32 * TN;
    const int tiles_m = (g.M + BM - 1) / BM;
    const int tiles_n = (g.N + BN - 1) / BN;
    const int grid = (tiles_m * tiles_n * splitk + 7) / 8 * 8;
    const size_t smem = (size_t)2 * (BM + BN) * BK * sizeof(bf16);
    static_assert((size_t)2 * (BM + BN) * BK * sizeof(bf16) >= 4 * EPI_WAVE_FLOATS * sizeof(float), "epilogue staging");
    static std::once_flag attr_once;          // one per instantiation
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&]() {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_kernel<TM, TN, BK, PF>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    });
    if (attr_err != hipSuccess || attributes_only()) return attr_err;
    const int group_m = 8;
    if (g_launch_note.on) snprintf(g_launch_note.kernel, sizeof(g_launch_note.kernel), "gemm_kernel<%d, %d, %d, %d>", TM, TN, BK, PF);
    hipLaunchKernelGGL((gemm_kernel<TM, TN, BK, PF>), dim3(grid), dim3(256), smem, s, g, tiles_m, tiles_n, group_m, splitk);
    return hipGetLastError();
}

template <int TM, int PF>
hipError_t launch_tn(const GemmArgs& g, int tn, int splitk, hipStream_t s) {
    switch (tn) {
        case 2: return launch_one<TM, 2, PF>(g, splitk, s);
        case 3: return launch_one<TM, 3, PF>(g, splitk, s);
        case 4: return launch_one<TM, 4, PF>(g, splitk, s);
        case 5: return launch_one<TM, 5, PF>(g, splitk, s);
        case 6: return launch_one<TM, 6, PF>(g, splitk, s);
    }
    if constexpr (PF == 2) {
        switch (tn) {
            case 7: return launch_one<TM, 7, PF>(g, splitk, s);
            case 8: return launch_one<TM, 8, PF>(g, splitk, s);
        }
    }
    return hipErrorInvalidValue;
}

// Configurations of gemm_alt64_kernel: waves on M and N, wave tile in 16-row and 16-column blocks, stages of A and W,
// ROLES, waves per SIMD the registers are budgeted for, workgroups per compute unit; then what a launch costs in
// microseconds:  c + rounds * (k tiles * a + b),  a = one k tile with the chip full of such tiles, b = prologue and
// epilogue of a tile, c = launch and drain.  `rounds` counts full rounds (one tile in every slot of the chip) and, for
// a last round that fills the share x of the slots, p + (1 - p) x of a round: less traffic and a higher clock, but no
// less latency (two workgroups per unit: p + s x up to x = 1/2, where a unit has one, q + (1 - q) x above).  Fitted to
// launches in a steady state (weights cold, the chip at its power limit) of 156 random shapes of 128 to 18 720 rows,
// K = 512 to 18 000: root mean square error 4 to 10 %, and the configuration picked is on average 0.5 % slower than the
// best of all of them.  256 x 256 fitted again since its loads go by scalar rows (a was 1.60): of 3000 random products of such
// models 132 take it now that did not; 44 of those measured are 2.8 % faster on average (6656 x 4096 x 12800 636 -> 588 us, 9504 x
// 3072 x 3072 152 -> 141; the worst 0.9 % slower, 14896 x 16000 x 5120 1882 -> 1896).
#define SDV2_TILE_CONFIGS(X)                                                                                  \
    X(1, 2, 4, 8, 4, 2, 3, false, 2, 1, 1.505f, 7.1f, 2.8f, 0.77f, 0.23f, 1.0f)   /* 256 x 256 */             \
    X(2, 2, 4, 6, 4, 2, 3, true, 2, 1, 1.156f, 4.3f, 3.4f, 0.68f, 0.32f, 1.0f)    /* 192 x 256 */             \
    X(3, 2, 2, 8, 6, 2, 3, false, 1, 1, 1.129f, 5.5f, 2.9f, 0.73f, 0.27f, 1.0f)   /* 256 x 192 */             \
    X(4, 4, 2, 4, 5, 3, 3, false, 2, 1, 1.031f, 4.4f, 3.2f, 0.71f, 0.29f, 1.0f)   /* 256 x 160 */             \
    X(5, 4, 2, 4, 4, 3, 3, false, 2, 1, 0.892f, 3.0f, 3.0f, 0.71f, 0.29f, 1.0f)   /* 256 x 128 */             \
    X(6, 2, 4, 6, 3, 2, 4, true, 2, 1, 0.940f, 3.6f, 3.1f, 0.75f, 0.25f, 1.0f)    /* 192 x 192 */             \
    X(7, 4, 2, 2, 6, 4, 4, true, 2, 1, 0.713f, 2.1f, 3.0f, 0.78f, 0.22f, 1.0f)    /* 128 x 192 */             \
    X(8, 4, 2, 2, 5, 4, 4, true, 2, 1, 0.638f, 1.9f, 2.8f, 0.82f, 0.18f, 1.0f)    /* 128 x 160 */             \
    X(9, 4, 2, 2, 4, 4, 5, true, 2, 1, 0.549f, 1.0f, 3.5f, 0.80f, 0.20f, 1.0f)    /* 128 x 128 */             \
    X(10, 4, 2, 2, 3, 5, 5, true, 2, 1, 0.472f, 0.8f, 3.8f, 0.80f, 0.20f, 1.0f)   /* 128 x 96 */              \
    X(11, 4, 2, 3, 4, 3, 4, true, 2, 1, 0.725f, 2.1f, 3.4f, 0.71f, 0.29f, 1.0f)   /* 192 x 128 */             \
    X(12, 2, 2, 4, 6, 2, 2, false, 2, 2, 1.339f, 2.7f, 2.0f, 0.64f, 0.20f, 0.85f) /* 128 x 192, two */        \
    X(13, 2, 2, 4, 2, 3, 3, false, 2, 2, 0.724f, 0.0f, 3.7f, 0.47f, 0.25f, 0.85f) /* 128 x 64, two */         \
    X(14, 2, 2, 2, 4, 3, 3, false, 2, 2, 0.731f, 0.0f, 3.7f, 0.48f, 0.27f, 0.95f) /* 64 x 128, two */         \
    X(15, 2, 2, 2, 3, 4, 4, false, 2, 2, 0.600f, 0.3f, 3.8f, 0.45f, 0.24f, 0.93f) /* 64 x 96, two */          \
    X(16, 2, 2, 2, 2, 5, 5, false, 2, 2, 0.482f, 0.0f, 3.8f, 0.48f, 0.18f, 0.95f) /* 64 x 64, two */          \
    X(17, 2, 2, 2, 1, 6, 6, false, 2, 2, 0.346f, 0.35f, 3.5f, 0.53f, 0.10f, 1.0f) /* 64 x 32, two */          \
    X(18, 2, 2, 1, 1, 8, 8, false, 2, 2, 0.245f, 1.09f, 3.14f, 0.53f, 0.19f, 1.0f)   /* 32 x 32, two */
constexpr int kTileConfigs = 18;

// A launch that gives each compute unit one workgroup of tiles that fit it twice has its weights fetched once in large pieces
// by workgroups in the second places, 32 KB each (64 KB of the largest: 256 workgroups at most), while its own begin: the k loop asks HBM for 128 bytes of every row at
// a time, from as many DRAM pages, which costs more than the bytes.  Weights from HBM without and with this (and from the
// memory-side cache): 1024 x 1536 x 1536 12.8 -> 10.7 us (10.5 and 10.3); 512 x 1536 x 1536 10.3 -> 8.0 (7.4 and 7.6);
// 1024 x 2048 x 2048 19.1 -> 16.3 (15.5 and 15.8); 1.3B step 6.18 -> 6.03 ms, prompt 487 -> 449 us.
// A workgroup of a larger tile has its unit to itself; fetches in front of its own loads, or in left-over units, gave nothing.
// More than 16 MB would take longer than the first k tiles they are to be ahead of; weights that are in the memory-side cache
// anyway (cold_weights) are left alone: 65 x 1280 x 1280, two products, 9.1 us without, 9.9 with.
constexpr size_t kMostOwnWeights = (size_t)16 << 20;
template <int PER_UNIT>
bool fetches_own_weights(const GemmArgs& g, int grid) {
    return PER_UNIT == 2 && g.cold_weights && grid <= kUnits &&
           (size_t)g.N * g.K * sizeof(bf16) * (g.w2 != nullptr ? 2 : 1) <= kMostOwnWeights;
}

void alt64_name(char* out, size_t cap, bool fetching, int wm, int wn, int tm, int tn, int nsa, int nsw, bool roles, int occ) {
    snprintf(out, cap, "gemm_%s_kernel<%d, %d, %d, %d, %d, %d, %s, %d>", fetching ? "fetching" : "alt64", wm, wn, tm, tn, nsa, nsw,
             roles ? "true" : "false", occ);
}

template <int WM, int WN, int TM, int TN, int NSA, int NSW, bool ROLES, int OCC, int PER_UNIT>
hipError_t launch_alt64(const GemmArgs& g, int splitk, hipStream_t s, const WarmArgs* side) {
    constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
    constexpr size_t smem = (size_t)(NSA * BM + NSW * BN) * 64 * sizeof(bf16);
    static_assert(smem * PER_UNIT <= 160 * 1024, "LDS stages exceed 160 KB");
    const int tiles_m = (g.M + BM - 1) / BM;
    const int tiles_n = (g.N + BN - 1) / BN;
    int grid = (tiles_m * tiles_n * splitk + 7) / 8 * 8;
    // one workgroup per slot of the chip, which then takes its tiles in turn.  A k part is a tile range of its own, and
    // the loads may not run past the next tile (k shorter than the ring): one tile per workgroup then.
    if (splitk == 1 && g.K / 64 > NSW && grid > kUnits * PER_UNIT) grid = kUnits * PER_UNIT;
    static std::once_flag attr_once;          // one per instantiation
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&]() {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_alt64_kernel<WM, WN, TM, TN, NSA, NSW, ROLES, OCC>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (attr_err == hipSuccess)
            attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_fetching_kernel<WM, WN, TM, TN, NSA, NSW, ROLES, OCC>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    });
    if (attr_err != hipSuccess || attributes_only()) return attr_err;
    // tile rows that share weight tiles: an XCD's 32 concurrent large tiles then cover 4 x 8 tiles, the shape with the
    // fewest distinct operand rows per k step
    const int group_m = BM >= 192 ? 4 : 8;
    WarmArgs warm;
    memset(&warm, 0, sizeof(warm));
    if (side != nullptr) warm = *side;
    if (fetches_own_weights<PER_UNIT>(g, grid)) {
        const unsigned pitch = (unsigned)g.K * 2u, columns = (pitch + 1023u) / 1024u;
        warm.ranges = g.w2 != nullptr ? 2 : 1;
        warm.range[0] = WarmRange{reinterpret_cast<const unsigned char*>(g.w), (unsigned)g.N, pitch, columns};
        if (g.w2 != nullptr) warm.range[1] = WarmRange{reinterpret_cast<const unsigned char*>(g.w2), (unsigned)g.N, pitch, columns};
        const size_t blocks = (size_t)warm.ranges * g.N * pitch / (32 * 1024);
        warm.blocks = blocks < kUnits ? (unsigned)blocks : kUnits;
    }
    if (g_launch_note.on) alt64_name(g_launch_note.kernel, sizeof(g_launch_note.kernel), warm.blocks > 0, WM, WN, TM, TN, NSA, NSW, ROLES, OCC);
    if (warm.blocks > 0)
        hipLaunchKernelGGL((gemm_fetching_kernel<WM, WN, TM, TN, NSA, NSW, ROLES, OCC>), dim3(grid + warm.blocks), dim3(64 * WM * WN), smem, s, g,
                           tiles_m, tiles_n, group_m, splitk, (unsigned)grid, warm);
    else
        hipLaunchKernelGGL((gemm_alt64_kernel<WM, WN, TM, TN, NSA, NSW, ROLES, OCC>), dim3(grid), dim3(64 * WM * WN), smem, s, g, tiles_m, tiles_n,
                           group_m, splitk);
    return hipGetLastError();
}

struct TileCost {
    int bm, bn, waves_n, per_unit;
    bool one_wave;                    // a SIMD holds a single wave
    float a, b, c, p, s, q;
};
const TileCost kCost[kTileConfigs + 1] = {
    {0, 0, 0, 0, false, 0, 0, 0, 0, 0, 0},
#define X(id, wm, wn, tm, tn, nsa, nsw, roles, occ, per_unit, a, b, c, p, s, q) {16 * tm * wm, 16 * tn * wn, wn, per_unit, occ == 1, a, b, c, p, s, q},
    SDV2_TILE_CONFIGS(X)
#undef X
};

hipError_t launch_tile_config(const GemmArgs& g, int id, int splitk, hipStream_t s, const WarmArgs* warm = nullptr) {
    if (!fits_32bit_offsets(g.M, g.N, g.K) || !operands_aligned(g)) return hipErrorInvalidValue;     // only reachable through the tuning override
    switch (id) {
#define X(id, wm, wn, tm, tn, nsa, nsw, roles, occ, per_unit, ...) \
    case id: return launch_alt64<wm, wn, tm, tn, nsa, nsw, roles, occ, per_unit>(g, splitk, s, warm);
        SDV2_TILE_CONFIGS(X)
#undef X
    }
    return hipErrorInvalidValue;
}

// Estimated microseconds of configuration `id` on an M x N output with `k_tiles` k tiles of 64 in each of `parts` parts.
float tile_cost(int id, int M, int N, float k_tiles, int parts) {
    const TileCost& t = kCost[id];
    const long long tiles = (long long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * parts;
    const int slots = kUnits * t.per_unit;
    const float full = (float)(tiles / slots), x = (float)(tiles % slots) / (float)slots;
    float last = 0.0f;
    if (x > 0.0f) last = (t.per_unit == 1 || x <= 0.5f) ? t.p + t.s * x : t.q + (1.0f - t.q) * x;
    return t.c + (full + last) * (k_tiles * t.a + t.b);
}

// The planner: the configuration and number of k parts with the smallest estimate among those that the call can run.  A k
// split pays for a second pass (4 us and its bytes at 3.9 TB/s); a residual epilogue gets back the LayerNorm that this pass
// forms (5 us).  Parts of at least 512, as many as the call's scratch holds (a tile picked for a split that is then not made
// is up to 1.8 times slower than the best whole one: 77 text tokens of 40 heads, 64 us a layer instead of 39), and at most
// 48 MiB of partial sums (long sums: below).  Up to 32 MiB they fit the entry point without a workspace; more than that has to
// be 1.5 % better by the estimate, which is careful: measured with cold weights, best within 32 MiB against the plan with 32
// to 48 MiB: 1024 x 3072 x 12288 87 -> 77 us, 1560 x 3072 x 12288 124 -> 120.
constexpr size_t kMaxPartialBytes = (size_t)48 << 20, kSmallPartialBytes = (size_t)32 << 20;
constexpr int kMaxParts = 6;
// Sums of more than 12 288 products take at least three parts where the scratch and 64 MiB hold them: the error of a sum
// grows with the root of its longest chain.  1024 x 5120 x 13824 (FFN-2 of the 14B block), relative error against 64 bits:
// whole 7.5e-7, two parts 5.2e-7, three 4.2e-7; 145, 128 and 139 us.
constexpr int kLongSum = 12288, kLongSumParts = 3;
constexpr size_t kMaxLongSumBytes = (size_t)64 << 20;

size_t most_partial_bytes(int K) { return K > kLongSum ? kMaxLongSumBytes : kMaxPartialBytes; }

// Parts of k (1: no split) that leave 512 of k to each and whose partial sums fit in `bytes` of scratch.
int most_parts(int M, int N, int K, size_t bytes) {
    const size_t cap = most_partial_bytes(K), fit = (bytes < cap ? bytes : cap) / ((size_t)M * N * sizeof(float));
    const int by_k = K / 512;
    int parts = fit < (size_t)kMaxParts ? (int)fit : kMaxParts;
    if (parts > by_k) parts = by_k;
    return parts < 1 ? 1 : parts;
}

// Estimated microseconds of configuration `id` for one or two products of a shape, split in `parts` parts of k.
float plan_cost(int id, int M, int N, int K, int epilogue, int parts, int products) {
    const bool residual = epilogue == kEpiGatedResidual || epilogue == kEpiResidual;
    float cost = tile_cost(id, M, N, (float)K / (64 * parts), parts * products);
    if (parts > 1) cost += 4.0f + (float)M * N * (4.0f * parts + (residual ? 8.0f : 2.0f)) / 3.9e6f - (residual ? 5.0f : 0.0f);
    // operands beyond the 256 MB memory-side cache: with a single wave per SIMD their latency shows (4 to 14 %)
    if (kCost[id].one_wave && ((size_t)M + (size_t)products * N) * K * sizeof(bf16) > ((size_t)240 << 20)) cost *= 1.07f;
    if (parts > 1 && (size_t)parts * M * N * sizeof(float) > kSmallPartialBytes) cost *= 1.015f;
    // An fp32 x beyond half of that cache is read and written again in HBM by the epilogue, which a single wave per SIMD hides
    // least of all (more loads of x in flight change nothing).  What the residual adds to the same product with a bf16 store, 256
    // x 256, 192 x 256, 256 x 192 and 256 x 160 tiles: 18720 x 5120 x 5120 110, 120, 159 and 131 us; 12480 x 5120 x 5120 85, 99,
    // 136 and 101; 8192 x 5120 x 5120 52, 51, 73 and 39; 8192 x 2560 x 2560 (x of 84 MB) 23, 16, 18 and 13.  The lines
    // alone put 256 x 192 (922 us) level with 256 x 256 and 192 x 256 (840 and 843) for the first.
    if (parts == 1 && residual && kCost[id].one_wave && (size_t)M * N * sizeof(float) > ((size_t)120 << 20)) cost += (float)M * N * 8.0f / 15e6f;
    return cost;
}

TilePlan search_plan(int M, int N, int K, int epilogue, int max_parts, int products) {
    TilePlan best{0, 0, 0, 1, 1};
    float best_cost = 1e30f;
    const int kParts[] = {1, 2, 3, 4, kMaxParts};
    const int min_parts = K > kLongSum && max_parts >= kLongSumParts ? kLongSumParts : 1;
    for (const int parts : kParts) {
        if (parts < min_parts) continue;
        if (parts > max_parts) break;
        for (int id = 1; id <= kTileConfigs; ++id) {
            const float cost = plan_cost(id, M, N, K, epilogue, parts, products);
            if (cost < best_cost) {
                best_cost = cost;
                best = TilePlan{0, 0, 0, id, parts};
            }
        }
    }
    return best;
}

// The plan of a call with `bytes` of scratch for partial sums; products = 2: two of the same A in one launch, which makes no
// split.  Kept for the shapes a thread has used last (a step asks for the same half dozen over and over; a search is 18 x 5
// estimates, about 2 us).
TilePlan plan_tiles(int M, int N, int K, int epilogue, size_t bytes, int products = 1) {
    if (!fits_32bit_offsets(M, N, K)) return plan_register_staged(M, N, K);
    struct Entry {
        int M, N, K, kind;
        TilePlan plan;
    };
    constexpr int kEntries = 64;
    static thread_local Entry cache[kEntries] = {};
    const int residual = epilogue == kEpiGatedResidual || epilogue == kEpiResidual ? 1 : 0;
    const int max_parts = products > 1 ? 1 : most_parts(M, N, K, bytes);
    const int kind = residual + 2 * products + 8 * max_parts;
    const uint32_t h = (uint32_t)M * 2654435761u ^ (uint32_t)N * 2246822519u ^ (uint32_t)K * 3266489917u ^ (uint32_t)kind;
    Entry& e = cache[(h ^ (h >> 16)) % kEntries];
    if (e.M != M || e.N != N || e.K != K || e.kind != kind) e = Entry{M, N, K, kind, search_plan(M, N, K, epilogue, max_parts, products)};
    return e.plan;
}

size_t scratch_bytes(const GemmArgs& g) { return g.splitk_partials == nullptr ? 0 : g.splitk_floats * sizeof(float); }

}  // namespace

// Plan override for tuning runs and tests, set through sdv2_tuning_set("gemm_tile", ...): "tm,tn[,pf[,splitk]]"
// picks a tile of the register-staged kernel, "d<id>[,splitk]" a configuration of gemm_alt64_kernel; an empty
// string or null clears it.  Not read from the environment: a production
// process cannot change a kernel plan by accident, and a launch costs no getenv.
static bool g_have_tile_override = false;
static TilePlan g_tile_override;

bool set_gemm_tile_override(const char* e) {
    if (!e || !*e) {
        g_have_tile_override = false;
        return true;
    }
    int a, b, d = 2;
    int dk = 1;
    if (sscanf(e, "d%d,%d", &a, &dk) >= 1 && a >= 1 && a <= kTileConfigs && dk >= 1 && dk <= 16) {
        g_tile_override = TilePlan{0, 0, 0, a, dk};
        g_have_tile_override = true;
        return true;
    }
    int k = 1;
    if (sscanf(e, "%d,%d,%d,%d", &a, &b, &d, &k) >= 2 && a >= 1 && a <= 2 && b >= 2 && b <= 8 &&
        (d == 2 || (d == 3 && b <= 6)) && k >= 1 && k <= 8) {
        g_tile_override = TilePlan{a, b, d, 0, k};
        g_have_tile_override = true;
        return true;
    }
    return false;
}

static thread_local bool g_attr_only = false;
void set_attributes_only(bool on) { g_attr_only = on; }
bool attributes_only() { return g_attr_only; }

static bool tile_override(TilePlan* p) {
    if (g_have_tile_override) *p = g_tile_override;
    return g_have_tile_override;
}

namespace {
// out = epilogue(sum of the k parts + bias), four columns per thread; the parts are added in k order.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs g, int splitk) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;      // over M * N / 4
    const size_t n4 = (size_t)(g.N >> 2);
    if (idx >= (size_t)g.M * n4) return;
    const int row = (int)(idx / n4);
    const int col = (int)(idx - (size_t)row * n4) * 4;
    const size_t o = (size_t)row * g.N + col;
    const size_t part = (size_t)g.M * g.N;
    f32x4 v = *reinterpret_cast<const f32x4*>(g.splitk_partials + o);
    for (int s = 1; s < splitk; ++s) v += *reinterpret_cast<const f32x4*>(g.splitk_partials + s * part + o);
    if (g.bias != nullptr) v += *reinterpret_cast<const f32x4*>(g.bias + col);
    if (g.epilogue == kEpiBias || g.epilogue == kEpiBiasGelu) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (bf16)(g.epilogue == kEpiBiasGelu ? gelu_tanh_f(v[e]) : v[e]);
        *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(g.out) + o) = w;
    } else {
        if (g.epilogue == kEpiGatedResidual) {
            const f32x4 ga = *reinterpret_cast<const f32x4*>(g.gate_a + col);
            const f32x4 gb = *reinterpret_cast<const f32x4*>(g.gate_b + (size_t)(row / g.rows_per_gate) * g.gate_b_stride + col);
            v *= (ga + gb);
        }
        float* xo = reinterpret_cast<float*>(g.out) + o;
        *reinterpret_cast<f32x4*>(xo) = *reinterpret_cast<const f32x4*>(xo) + v;
    }
}
}  // namespace

namespace {
// The same sum of the k parts for a residual epilogue whose result is LayerNorm-ed next: a workgroup of four waves
// owns a row, adds the parts in k order, applies bias, gate and residual, stores the new fp32 row, and normalises it
// from the registers: one launch and one read of x less than reduce + LayerNorm.  (One row per workgroup: the pass
// reads splitk + 1 fp32 rows per output row, and with fewer, fatter workgroups it ran at 2.5 TB/s.)
// On one chunk the pass is a chain of latencies, so the loads stand in straight-line code: behind a branch (columns past the
// end) or in a loop over the parts each waits for the one before.  Columns past the end fetch the last piece, which is not
// used; gate and modulation are there or not at compile time.  Rows of up to 3072 columns fetch everything at once; wider
// ones form the new row first and fetch the LayerNorm's rows under its sums, so that two to four workgroups fit a unit.
// Measured, behind branches -> everything at once at every width, absent operands too -> this: 512 x 5120 in three parts 14.7
// -> 13.0 -> 12.2 us, 1024 x 5120 in three 23.2 -> 23.3 -> 21.6, 1024 x 4096 in four 18.8 -> 27.2 -> 19.1, 1024 x 6144 in three
// 23.9 -> 33.8 -> 24.0, 1024 x 1536 in four 8.9 -> 9.1 -> 8.4; at most 5 % slower than the first at any width, rows and parts that
// are planned.
// SP: parts, known to the compiler where the planner picks them often (0: any number, a part of the whole row at a time).
template <int NV, int SP, bool GATED, bool MODULATED>
__global__ __launch_bounds__(256) void splitk_reduce_ln_kernel(GemmArgs g, int splitk, LnArgs ln) {
    __shared__ float part[4][2];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int t = threadIdx.x;
    const int row = blockIdx.x;
    const int nvec = g.N >> 2;
    const size_t plane = (size_t)g.M * g.N;
    float* xrow = reinterpret_cast<float*>(g.out) + (size_t)row * g.N;
    const float* prow = g.splitk_partials + (size_t)row * g.N;
    const int stream = row / g.rows_per_gate;
    const int ln_stream = row / ln.rows_per_stream;
    const float pivot = xrow[0];                          // a value near the row's mean: read before the row is rewritten
    const bool has_bias = g.bias != nullptr;
    const float* const bias = has_bias ? g.bias : ln.scale_a;
    constexpr int kEarly = SP > 0 ? SP : 1;
    constexpr bool kLate = NV > 3;                        // the LayerNorm's rows under the sums
    f32x4 p[NV][kEarly], xv[NV];
    int col[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = col[i] = min(t + 256 * i, nvec - 1) * 4;
#pragma unroll
        for (int sp = 0; sp < kEarly; ++sp) p[i][sp] = *reinterpret_cast<const f32x4*>(prow + sp * plane + c);
        xv[i] = *reinterpret_cast<const f32x4*>(xrow + c);
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x4 ba[NV], ga[NV];
    auto load_epilogue = [&]() {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            ba[i] = *reinterpret_cast<const f32x4*>(bias + col[i]);
            if (GATED)
                ga[i] = *reinterpret_cast<const f32x4*>(g.gate_a + col[i]) +
                        *reinterpret_cast<const f32x4*>(g.gate_b + (size_t)stream * g.gate_b_stride + col[i]);
        }
    };
    f32x4 sca[NV], sha[NV], scb[NV], shb[NV];
    auto load_norm = [&]() {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            sca[i] = *reinterpret_cast<const f32x4*>(ln.scale_a + col[i]);
            sha[i] = *reinterpret_cast<const f32x4*>(ln.shift_a + col[i]);
            if (MODULATED) {
                scb[i] = *reinterpret_cast<const f32x4*>(ln.scale_b + (size_t)ln_stream * ln.b_stride + col[i]);
                shb[i] = *reinterpret_cast<const f32x4*>(ln.shift_b + (size_t)ln_stream * ln.b_stride + col[i]);
            }
        }
    };
    if (!kLate) {
        load_epilogue();
        load_norm();
    }
    if constexpr (SP == 0) {
        for (int sp = 1; sp < splitk; ++sp) {
            f32x4 next[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) next[i] = *reinterpret_cast<const f32x4*>(prow + sp * plane + col[i]);
#pragma unroll
            for (int i = 0; i < NV; ++i) p[i][0] += next[i];
        }
    }
    if (kLate) load_epilogue();
    f32x4 v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
#pragma clang fp contract(off)                            // gate times sum is rounded before x joins, as in the other passes
        f32x4 acc = p[i][0];
#pragma unroll
        for (int sp = 1; sp < kEarly; ++sp) acc += p[i][sp];
        acc = has_bias ? acc + ba[i] : acc;
        acc = GATED ? acc * ga[i] : acc;
        v[i] = xv[i] + acc;
        if (kLate) asm volatile("" : "+v"(v[i]));         // formed here, not where it is stored: its operands' registers are free
    }
    if (kLate) {                                          // on its way under the sums
        __builtin_amdgcn_sched_barrier(0);
        load_norm();
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();                                      // every thread of the row has read the pivot before x changes
    float sum = 0.0f, sq = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = t + 256 * i;
        if (idx < nvec) {
            *reinterpret_cast<f32x4*>(xrow + idx * 4) = v[i];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d = v[i][e] - pivot;
                sum += d;
                sq += d * d;
            }
        }
    }
    sum = wave_sum(sum);
    sq = wave_sum(sq);
    if (lane == 0) {
        part[wave][0] = sum;
        part[wave][1] = sq;
    }
    __syncthreads();
    sum = (part[0][0] + part[1][0]) + (part[2][0] + part[3][0]);
    sq = (part[0][1] + part[1][1]) + (part[2][1] + part[3][1]);
    const float inv_c = 1.0f / (float)g.N;
    float dmean = sum * inv_c;
    float var = fmaxf(sq * inv_c - dmean * dmean, 0.0f);
    float mean = pivot + dmean;
    // The pivot is of the row before the update.  Where the update has moved the mean far from it, the variance is the small
    // difference of two large numbers: form it again around the mean.  The same decision in every thread of the row.
    if (dmean * dmean > 256.0f * var) {
        __syncthreads();                                  // part[] has been read
        sum = 0.0f;
        sq = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (t + 256 * i < nvec) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d = v[i][e] - mean;
                    sum += d;
                    sq += d * d;
                }
            }
        }
        sum = wave_sum(sum);
        sq = wave_sum(sq);
        if (lane == 0) {
            part[wave][0] = sum;
            part[wave][1] = sq;
        }
        __syncthreads();
        dmean = ((part[0][0] + part[1][0]) + (part[2][0] + part[3][0])) * inv_c;
        var = fmaxf(((part[0][1] + part[1][1]) + (part[2][1] + part[3][1])) * inv_c - dmean * dmean, 0.0f);
        mean += dmean;
    }
    const float rstd = rsqrtf(var + ln.eps);
    bf16* op = ln.out + (size_t)row * g.N;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = t + 256 * i;
        if (idx < nvec) {
            const f32x4 sc = MODULATED ? (sca[i] + scb[i]) + 1.0f : sca[i], sh = MODULATED ? sha[i] + shb[i] : sha[i];
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)((v[i][e] - mean) * rstd * sc[e] + sh[e]);
            *reinterpret_cast<bf16x4*>(op + idx * 4) = o;
        }
    }
}
}  // namespace

// The pass above for rows of N columns (null: too many), NV = float4 values per thread.
typedef void (*ReduceLnKernel)(GemmArgs, int, LnArgs);
template <int NV, bool GATED, bool MODULATED>
static ReduceLnKernel reduce_ln_kernel_of_parts(int splitk) {
    switch (splitk) {
        case 2: return splitk_reduce_ln_kernel<NV, 2, GATED, MODULATED>;
        case 3: return splitk_reduce_ln_kernel<NV, 3, GATED, MODULATED>;
        case 4: return splitk_reduce_ln_kernel<NV, 4, GATED, MODULATED>;
    }
    return splitk_reduce_ln_kernel<NV, 0, GATED, MODULATED>;
}
template <bool GATED, bool MODULATED>
static ReduceLnKernel reduce_ln_kernel(int N, int splitk) {
    switch ((N + 1023) / 1024) {
        case 1: return reduce_ln_kernel_of_parts<1, GATED, MODULATED>(splitk);
        case 2: return reduce_ln_kernel_of_parts<2, GATED, MODULATED>(splitk);
        case 3: return reduce_ln_kernel_of_parts<3, GATED, MODULATED>(splitk);
        case 4: return reduce_ln_kernel_of_parts<4, GATED, MODULATED>(splitk);
        case 5: return reduce_ln_kernel_of_parts<5, GATED, MODULATED>(splitk);
        case 6: return splitk_reduce_ln_kernel<6, 0, GATED, MODULATED>;
        case 7: return splitk_reduce_ln_kernel<7, 0, GATED, MODULATED>;
        case 8: return splitk_reduce_ln_kernel<8, 0, GATED, MODULATED>;
    }
    return nullptr;
}

// The plan of a call: two products of one launch (w2) make no split.
static TilePlan plan_of(const GemmArgs& g) {
    TilePlan p = !operands_aligned(g)  ? plan_register_staged(g.M, g.N, g.K)
                 : g.w2 != nullptr     ? plan_tiles(g.M, g.N, g.K, g.epilogue, 0, 2)
                                       : plan_tiles(g.M, g.N, g.K, g.epilogue, scratch_bytes(g));
    tile_override(&p);
    return p;
}

// Parts of k the plan can really use for this problem and scratch (1: no split).
static int usable_splitk(const GemmArgs& g, const TilePlan& p) {
    if (p.splitk <= 1 || g.splitk_partials == nullptr) return 1;
    int splitk = p.splitk;
    if (splitk > g.K / 128) splitk = g.K / 128;                 // at least two k tiles per part
    const size_t fit = g.splitk_floats / ((size_t)g.M * g.N);   // parts that the scratch holds
    if ((size_t)splitk > fit) splitk = (int)fit;
    return splitk < 2 ? 1 : splitk;
}

// part 0: the whole product; 1: only the kernel on the matrix cores; 2: only the pass that adds the k parts (nothing
// when the plan does not split).  The benchmark times the two parts separately.
static hipError_t launch_gemm_impl(const GemmArgs& g, const LnArgs* ln, bool* ln_done, hipStream_t s, int part = 0, const WarmArgs* side = nullptr) {
    if (g.w2 != nullptr) {
        const TilePlan p2 = plan_of(g);
        if (p2.dma) return launch_tile_config(g, p2.dma, 2, s, side);
        GemmArgs one = g;
        one.w2 = nullptr;
        const hipError_t e1 = launch_gemm_impl(one, nullptr, nullptr, s);
        if (e1 != hipSuccess) return e1;
        one.w = g.w2;
        one.bias = g.bias2;
        one.out = g.out2;
        return launch_gemm_impl(one, nullptr, nullptr, s);
    }
    const TilePlan p = plan_of(g);
    const int splitk = usable_splitk(g, p);
    hipError_t e = hipSuccess;
    if (part != 2) {
        if (p.dma) e = launch_tile_config(g, p.dma, splitk, s, side);
        else if (p.pf == 3) e = p.tm == 1 ? launch_tn<1, 3>(g, p.tn, splitk, s) : launch_tn<2, 3>(g, p.tn, splitk, s);
        else e = p.tm == 1 ? launch_tn<1, 2>(g, p.tn, splitk, s) : launch_tn<2, 2>(g, p.tn, splitk, s);
    }
    if (e != hipSuccess || splitk == 1 || attributes_only() || part == 1) return e;
    if (ln != nullptr && (g.epilogue == kEpiGatedResidual || g.epilogue == kEpiResidual)) {
        const bool gated = g.epilogue == kEpiGatedResidual, modulated = ln->scale_b != nullptr;
        const ReduceLnKernel kernel = gated ? (modulated ? reduce_ln_kernel<true, true>(g.N, splitk) : reduce_ln_kernel<true, false>(g.N, splitk))
                                            : (modulated ? reduce_ln_kernel<false, true>(g.N, splitk) : nullptr);     // no block asks for the last
        if (kernel != nullptr) {
            hipLaunchKernelGGL(kernel, dim3(g.M), dim3(256), 0, s, g, splitk, *ln);
            *ln_done = true;
            return hipGetLastError();
        }
    }
    const size_t n = (size_t)g.M * (g.N >> 2);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, splitk);
    return hipGetLastError();
}

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) { return launch_gemm_impl(g, nullptr, nullptr, s); }

// Name of the kernel instantiation the plan picks for a shape, spelled as a profiler prints it.
void gemm_plan_name(int M, int N, int K, int epilogue, char* out, size_t cap) {
    TilePlan p = plan_tiles(M, N, K, epilogue, most_partial_bytes(K));
    tile_override(&p);
    switch (p.dma) {
#define X(id, wm, wn, tm, tn, nsa, nsw, roles, occ, ...)                                                                 \
    case id:                                                                                                             \
        alt64_name(out, cap, false, wm, wn, tm, tn, nsa, nsw, roles, occ);                                               \
        return;
        SDV2_TILE_CONFIGS(X)
#undef X
    }
    snprintf(out, cap, "gemm_kernel<%d, %d, 64, %d>", p.tm, p.tn, p.pf);
}

void gemm_plan(int M, int N, int K, int epilogue, int products, size_t bytes, int* tile, int* parts, float* us) {
    TilePlan p = plan_tiles(M, N, K, epilogue, bytes, products);
    tile_override(&p);
    *tile = p.dma;
    *parts = p.splitk;
    *us = p.dma ? plan_cost(p.dma, M, N, K, epilogue, p.splitk, products) : 0.0f;
}

hipError_t launch_gemm_then_layernorm(const GemmArgs& g, const LnArgs& ln, bool* ln_done, hipStream_t s, int part) {
    *ln_done = false;
    return launch_gemm_impl(g, &ln, ln_done, s, part);
}

hipError_t launch_gemm_part(const GemmArgs& g, hipStream_t s, int part, const WarmArgs* warm) {
    return launch_gemm_impl(g, nullptr, nullptr, s, part, warm);
}

IdleUnits gemm_idle_units(const GemmArgs& g) {
    const TilePlan p = plan_of(g);
    IdleUnits idle{0, 8, 0.0f};
    if (!p.dma || kCost[p.dma].per_unit != 1) return idle;
    const TileCost& t = kCost[p.dma];
    const int parts = usable_splitk(g, p), tiles = ((g.M + t.bm - 1) / t.bm) * ((g.N + t.bn - 1) / t.bn) * parts;
    const int grid = (tiles + 7) / 8 * 8;
    if (grid < kUnits) idle.blocks = (unsigned)(kUnits - grid);
    idle.waves = t.one_wave ? 4 : 8;
    idle.us = tile_cost(p.dma, g.M, g.N, (float)g.K / (64 * parts), parts);
    return idle;
}

bool gemm_fetches_own_weights(const GemmArgs& g) {
    const TilePlan p = plan_of(g);
    if (!p.dma || kCost[p.dma].per_unit != 2) return false;
    const TileCost& t = kCost[p.dma];
    return fetches_own_weights<2>(g, ((g.M + t.bm - 1) / t.bm * ((g.N + t.bn - 1) / t.bn) * usable_splitk(g, p) + 7) / 8 * 8);
}

// One sum per row and wave column, which is how the epilogue's lanes hold them.
int gemm_square_pieces(const GemmArgs& g) {
    const TilePlan p = plan_of(g);
    if (!p.dma || usable_splitk(g, p) > 1) return 0;
    return (g.N + kCost[p.dma].bn - 1) / kCost[p.dma].bn * kCost[p.dma].waves_n;
}

hipError_t launch_gemm_gain_squares(const GemmArgs& g, hipStream_t s) {
    const TilePlan p = plan_of(g);
    GemmArgs a = g;
    a.epilogue = kEpiGainSquares;
    return launch_tile_config(a, p.dma, 1, s);
}

bool gemm_splits_k(const GemmArgs& g) {
    return usable_splitk(g, plan_of(g)) > 1;
}

size_t gemm_splitk_floats_bound(int M, int N, int K) {
    const size_t most = (size_t)kMaxParts * M * N, cap = most_partial_bytes(K) / sizeof(float);
    return most < cap ? most : cap;
}

size_t gemm_splitk_floats(int M, int N, int K, int epilogue) {
    TilePlan p = plan_tiles(M, N, K, epilogue, most_partial_bytes(K));
    tile_override(&p);
    if (p.splitk <= 1) return 0;
    return (size_t)p.splitk * M * N;
}

}  // namespace sdv2

