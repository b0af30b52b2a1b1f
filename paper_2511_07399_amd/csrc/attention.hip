// Exact attention of a chunk's queries over a prefix of cache slots, flash style (online softmax,
// no score matrix in memory), for gfx950.
//
// This is the "4 b L_q L_kv C" term of the per-layer cost in Appendix B of the paper; the paper runs
// it with a FlashAttention kernel (Section 4.1) over the sink + rolling-window cache (Appendix D).
// Because resident tokens always occupy the slot prefix [0, kv_len) of the ring layout and softmax
// attention does not depend on the order of the keys, the kernel scans physical slots in order and
// needs no [sink | window] segment logic.  The same kernel serves the text cross-attention.
//
// Design
//   * Workgroup = 4 waves = 128 queries of one (stream, head); each wave owns 32 queries; two workgroups
//     per compute unit.
//   * Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: keys are the rows,
//     queries the columns, so a lane (column = lane % 32) owns one query: its row maximum and row sum
//     live in that lane and its partner lane + 32, and the accumulator of S^T is already in the
//     register layout that the B operand of the second product O^T = V^T P^T wants.  No LDS round
//     trip for P.
//   * That needs V^T tiles with keys contiguous, which is why the cache stores values transposed
//     ([head][128][cap]); inside every group of 16 slots the cache swaps the middle two groups of four
//     (vt_column), which is the order in which the S^T accumulator holds its keys, so a V^T fragment is one
//     16-byte LDS read.  K tiles are contiguous 16 KB blocks of the [head][cap][128] key cache.
//   * K and V^T tiles of 64 keys go global -> LDS directly (global_load_lds_dwordx4), two stages each.  The
//     LDS swizzle is applied on the global side: K rows (256 B) XOR the 16-byte chunk index with row % 16,
//     V^T rows (128 B) with (row / 2) % 8, so that fragment reads are conflict free on the 64-bank LDS.
//   * The loop is software pipelined inside a wave: while the vector unit runs the softmax of tile t, the
//     matrix unit computes S^T of tile t + 1; the P V product of tile t follows.  The softmax costs about
//     as many vector cycles as the tile costs matrix cycles, so without this overlap (and that between
//     the two workgroups of a unit) the matrix unit idles half of the time.
//   * The exponents' reference point of a query trails its running maximum loosely instead of tracking it: the
//     steady-state loop forms no row maximum and rescales nothing; a sum of exponentials that leaves the range
//     sends the wave to a slow path that moves the reference point (it cancels in O / l).
//   * What a workgroup does before its first tile is a chain of latencies that a launch of a few tiles consists of: the
//     divisions that number the workgroups are products with the launcher's reciprocals (five in software took 1.5 us), the
//     arguments come in two batches, the queries pass through LDS (as fragments straight from memory they are 64 loads of
//     32 pieces of 32 bytes, and the first tiles queue behind them), and the first scores wait for the first K tile alone.
//     Queries that do not start at a multiple of 16 bytes are such fragments still: a direct load needs the multiple.
//     From the start to the first scores 5.6 -> 3.6 us; text cross-attention of the 1.3B chunk 13.0 -> 10.5 us, of the 14B
//     chunk 25 -> 21 us.  Outputs leave in pieces of 16 bytes.
//   * A query row's RMSNorm factor is one number, so it joins the scale of the query's scores (query_scale) instead of a pass
//     over the rows: the projection in front leaves gain times q and sums of squares, fetched under the first key tile.  One
//     launch of 4.5 us (1.3B chunk) to 68 us (480p batch of the 14B model) less per block, and one rounding less: the
//     branch's error against 64 bits 4.4e-3 -> 4.1e-3.
//   * Skinny launches (few query tiles x heads) split the key range over several workgroups, which
//     write normalised partial outputs with their (max, sum); a small kernel merges them.
#include "attention_ranges.h"
#include "common.h"

#include <stdio.h>
#include <stdlib.h>

#include <mutex>
#include <type_traits>

namespace sdv2 {

namespace {

constexpr int KT = 64;        // keys per tile
constexpr float kMaxSlack = 8.0f;   // log2 units within which a query's exponent reference is left where it is
constexpr float kNoKey = -1.0e30f;  // reference point of a query that has seen no key yet (key-split form)
constexpr float kSumLimit = 16384.0f;   // a lane's sum of p over one tile (at most 32 keys) beyond this: move the reference
constexpr int D = kHeadDim;
constexpr int K_TILE_BYTES = KT * D * 2;
constexpr int V_TILE_BYTES = D * KT * 2;

// max of three with one instruction and no NaN canonicalisation of the operands (scores are never NaN for
// valid slots; masked ones are -inf)
__device__ __forceinline__ float max3_f32(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

__device__ __forceinline__ float max2_f32(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// max of x over the lane pair (l, l ^ 32): one swap of the two 32-lane halves on the vector unit (a shuffle
// through the LDS crossbar would put its latency on the path to the exponentials)
__device__ __forceinline__ float max_xor32(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return max2_f32(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Makes the compiler hold the fragments in registers at this point of the program (an empty statement that claims to
// read and write them): conversions to bf16 cannot be moved past it.
template <int N>
__device__ __forceinline__ void pin_fragments(bf16x8 (&f)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(f[i]));
}

typedef __attribute__((address_space(3))) void* lds_void_ptr;
__device__ __forceinline__ void load_to_lds_b128(const void* src, void* dst) {
    __builtin_amdgcn_global_load_lds(src, (lds_void_ptr)dst, 16, 0, 0);
}

// Resident keys of stream b.  Read through the scalar cache: as a vector load it would be waited for together with the queries.
__device__ __forceinline__ int resident_keys(const AttnArgs& a, int b) {
    typedef const __attribute__((address_space(4))) int* scalar_int_ptr;
    if (a.desc != nullptr) return ((scalar_int_ptr) reinterpret_cast<uintptr_t>(a.desc->kv_len))[b];
    return a.kv_len[b];
}

// What a workgroup needs of its stream, requested in one batch.
struct StreamKeys {
    const bf16 *k, *vt;
    int cap, kv_len;
};
__device__ __forceinline__ StreamKeys stream_keys(const AttnArgs& a, int b) {
    StreamKeys s;
    s.k = a.k[b];
    s.vt = a.vt[b];
    s.cap = a.cap[b];
    s.kv_len = resident_keys(a, b);
    asm volatile("" ::"s"(s.k), "s"(s.vt), "s"(s.cap), "s"(s.kv_len));
    return s;
}

// Two groups of four channels of a query as bf16: a lane has channels 4 lh .. + 3 of two blocks of eight; the halves of the
// wave trade words so that each lane stores eight channels in a row (lanes < 32 the first block, the others the second).
__device__ __forceinline__ uint4 eight_channels(const bf16x4& lo, const bf16x4& hi) {
    const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
    const auto x = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
    return uint4{x[0], y[0], x[1], y[1]};
}

// Query tile, head and stream / split of a workgroup.  Workgroups are handed to the eight XCDs in turn; they are renumbered
// so that each XCD (its own L2) works through a contiguous run of (query tile, head, stream / split) triples, query tile
// fastest: the workgroups that share a head's K and V then sit behind the same L2.
__device__ __forceinline__ void locate(const AttnArgs& a, int& qt, int& h, int& bz) {
    // every argument that the first addresses need is requested at once: a scalar load that misses takes 0.2 to 0.5 us
    const FastDiv by_q_tiles = a.by_q_tiles, by_heads = a.by_heads;
    const unsigned n_wg = a.n_wg;
    asm volatile("" ::"s"(a.q), "s"(a.L), "s"(a.H), "s"(a.splits), "s"(a.desc), "s"(n_wg), "s"(by_q_tiles.d), "s"(by_q_tiles.m), "s"(by_heads.d),
                 "s"(by_heads.m));
    const unsigned flat = blockIdx.x, xcd = flat & 7u, per = n_wg >> 3, rem = n_wg & 7u;
    const unsigned logical = xcd * per + min(xcd, rem) + (flat >> 3);
    const unsigned rest = divide(logical, by_q_tiles), z = divide(rest, by_heads);
    qt = (int)(logical - rest * by_q_tiles.d);
    h = (int)(rest - z * by_heads.d);
    bz = (int)z;
}

// Loads of N groups of four query rows (1 KB each) to a stage whose row 0 is query q0 of the chunk, from row `first` on (past
// the chunk's end: its last query).  Row r of the stage holds chunk c at position c ^ (r % 16), as the K rows do.
template <int N>
__device__ __forceinline__ void load_queries(const AttnArgs& a, int b, int h, int q0, int first, int lane, unsigned char* stage, int C) {
    const unsigned char* src = reinterpret_cast<const unsigned char*>(a.q + (size_t)(unsigned)b * (unsigned)a.L * (unsigned)C + h * D);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int r = first + 4 * i + (lane >> 4);
        const size_t row = (unsigned)min(q0 + r, a.L - 1);
        load_to_lds_b128(src + row * (unsigned)(2 * C) + (((lane & 15) ^ (r & 15)) << 4), stage + (first + 4 * i) * 256);
    }
}
__device__ __forceinline__ void read_queries(bf16x8 (&qf)[D / 16], const unsigned char* stage, int l31, int lh) {
#pragma unroll
    for (int s = 0; s < D / 16; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(stage + l31 * 256 + (((2 * s + lh) ^ (l31 & 15)) << 4));
}

// The same fragments by ordinary vector loads, good for any address of a bf16.
__device__ __forceinline__ void fetch_queries(bf16x8 (&qf)[D / 16], const AttnArgs& a, size_t q_row, int h, int lh, int C) {
    const bf16* qp = a.q + q_row * C + h * D + lh * 8;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qp + s * 16);
}

// Scale of a query's scores: the softmax's, times the factor of the query's RMSNorm where that is still to be divided out.
// The two lanes of a query fetch half of the row's sums each, sixteen at a time (coalesced: rows are next to each other).
__device__ __forceinline__ float query_scale(const AttnArgs& a, float scale_log2e, size_t q_row, int lh) {
    if (a.q_squares == nullptr) return scale_log2e;
    const size_t rows = (size_t)(unsigned)a.B * (unsigned)a.L;
    const float* p = a.q_squares + q_row;
    float sum = 0.0f;
    for (int first = 0; first < a.q_pieces; first += 32) {
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = p[(unsigned)min(first + 2 * i + lh, a.q_pieces - 1) * rows];
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += first + 2 * i + lh < a.q_pieces ? v[i] : 0.0f;
    }
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
    sum = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    return scale_log2e * rsqrtf(sum / (float)(a.H * D) + a.q_eps);
}

// A row whose sum of squares is beyond fp32 has the factor 0: its norm is the zero row (not a number where q is infinite).  With
// a scale of 0 its masked scores, -inf, would be 0 x inf; so the queries become that row and keep the softmax's scale.
// True for a wave that has such a query: its scores are to be formed again.
__device__ __forceinline__ bool zero_queries(bf16x8 (&qf)[D / 16], float& scale, float softmax_scale) {
    const bool zero = scale == 0.0f;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(zero) == 0, 1)) return false;
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[s][e] = zero ? (bf16)((float)qf[s][e] * 0.0f) : qf[s][e];
    scale = zero ? softmax_scale : scale;
    return true;
}

constexpr int kNoMemory = 1;             // sched_barrier: instructions without memory access may cross

// STAGED: the queries go through LDS by direct loads, which need a multiple of 16 bytes.
template <int NW, bool STAGED>
__device__ __forceinline__ void attention_body(const AttnArgs& a, float softmax_scale) {
    constexpr int QT = 32 * NW;                   // queries per workgroup: one 32-query block per wave
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    unsigned char* const k_stage = smem_raw;                          // [2][64 keys][256 B]
    unsigned char* const v_stage = smem_raw + 2 * K_TILE_BYTES;       // [2][128 d][128 B]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31;
    const int lh = lane >> 5;

    int qt, h, bz;
    locate(a, qt, h, bz);
    const int b = a.splits == 1 ? bz : bz / a.splits;
    const int split = bz - b * a.splits;
    const int C = a.H * D;

    const StreamKeys keys = stream_keys(a, b);
    const int cap = keys.cap, kv_len = keys.kv_len;
    const KeyTiles part = key_tiles(kv_len, KT, split, a.splits);
    const int t0 = part.first, t_full = part.full, t1 = part.end;     // with few keys a part may be empty

    // ---- this lane's query (column of S^T) and its row.  Formed anew where they are needed, in front of the loop, for the
    // scale and at the end: kept across the loop they are spilled (256 registers), and the reloads wait for the tile loads.
    auto own_lane = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));
        return t & 63;
    };
    auto query_in_chunk = [&]() { return qt * QT + wave * 32 + (own_lane() & 31); };
    auto row_of = [&](int in_chunk) { return (size_t)(unsigned)b * (unsigned)a.L + (unsigned)min(in_chunk, a.L - 1); };

    // ---- The wave's 32 queries, through LDS (fetched as fragments they would be 8 loads of 32 pieces of 32 bytes each).  Eight
    // waves: behind the stages.  Four waves, two workgroups per unit: in the second stages, which are free until then.
    unsigned char* const q_stage =
        (NW == 8 ? smem_raw + 2 * (K_TILE_BYTES + V_TILE_BYTES) + wave * 8192 : (wave < 2 ? k_stage + K_TILE_BYTES : v_stage + V_TILE_BYTES) + (wave & 1) * 8192);
    bf16x8 qf[D / 16];           // this lane's query: its eight d-step fragments
    if (STAGED) load_queries<8>(a, b, h, qt * QT + wave * 32, 0, lane, q_stage, C);
    else fetch_queries(qf, a, row_of(query_in_chunk()), h, lh, C);

    // ---- direct loads.  A wave load fills 1 KB of LDS in lane order: 4 K rows or 8 V^T rows.  Wave w issues
    // loads w, w + NW, ... of each tile; the XOR term of a lane's chunk is the same for all of them.
    const unsigned char* kbase = reinterpret_cast<const unsigned char*>(keys.k + (size_t)h * cap * D);
    const unsigned char* vbase = reinterpret_cast<const unsigned char*>(keys.vt + (size_t)h * D * cap);
    constexpr int LPT = 16 / NW;                  // wave loads per K tile and per V^T tile for each wave
    const int k_row = 4 * wave + (lane >> 4);                                     // + 4 NW i
    const uint32_t k_off = (uint32_t)k_row * 256u + (uint32_t)(((lane & 15) ^ (k_row & 15)) * 16);
    const int v_row = 8 * wave + (lane >> 3);                                     // + 8 NW i
    const size_t v_off = (size_t)v_row * cap * 2 + (size_t)(((lane & 7) ^ ((v_row >> 1) & 7)) * 16);
    auto load_k = [&](int t, int stage) {
        const unsigned char* src = kbase + (size_t)t * K_TILE_BYTES + k_off;
        unsigned char* dst = k_stage + stage * K_TILE_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < LPT; ++i) load_to_lds_b128(src + i * (NW * 1024), dst + i * (NW * 1024));
    };
    auto load_v = [&](int t, int stage) {
        const unsigned char* src = vbase + (size_t)t * (KT * 2) + v_off;
        unsigned char* dst = v_stage + stage * V_TILE_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < LPT; ++i) load_to_lds_b128(src + (size_t)i * (8 * NW) * cap * 2, dst + i * (NW * 1024));
    };
    // Slots past kv_len may hold anything (NaN included) and 0 x NaN is not 0: blank them in the staged V^T tile.
    auto blank_v_tail = [&](int t, int stage) {
        const int n_valid = kv_len - t * KT;
        bf16* sv = reinterpret_cast<bf16*>(v_stage + stage * V_TILE_BYTES);
        for (int idx = tid; idx < D * 8; idx += 64 * NW) {
            const int row = idx >> 3, p = idx & 7;
            const int c = p ^ ((row >> 1) & 7);
            bf16x8 v = *reinterpret_cast<bf16x8*>(sv + row * KT + p * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int u = 8 * c + e;                                          // stored column
                const int slot = (u & ~12) | ((u & 4) << 1) | ((u & 8) >> 1);     // slot it holds (vt_column is an involution)
                if (slot >= n_valid) v[e] = (bf16)0.0f;
            }
            *reinterpret_cast<bf16x8*>(sv + row * KT + p * 8) = v;
        }
    };

    f32x16 o_acc[D / 32];
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o_acc[i][r] = 0.0f;
    float m_run = -INFINITY;     // reference point of this query's exponents: within kMaxSlack below the running maximum of its scaled (log2-domain) scores
    float l_run = 0.0f;          // this lane's share of the running sum

    // Half of S^T of the tile in stage sk: d steps 4 half .. 4 half + 3 of both 32-key blocks.  The eight K
    // fragments are read first, the MFMAs alternate between the two accumulators (a dependent MFMA would
    // wait 12 clocks longer for its predecessor).
    auto qk_half = [&](f32x16 (&s)[2], const unsigned char* sk, int half, auto&& after_reads) {
        if (half == 0) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kb][r] = 0.0f;
        }
        bf16x8 kf[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                kf[i][kb] = *reinterpret_cast<const bf16x8*>(sk + (kb * 32 + l31) * 256 +
                                                             (((2 * (4 * half + i) + lh) ^ (l31 & 15)) << 4));
        after_reads();
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i][kb], qf[4 * half + i], s[kb], 0, 0, 0);
    };
    auto nothing = []() {};

    auto wait_loads = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); };       // vmcnt(0) only
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    float scale_log2e = softmax_scale;
    f32x16 s_a[2], s_b[2];
    // one tile: s_cur holds S^T of tile t; S^T of tile t + 1 is formed into s_nxt on the way
    // (tail: compile-time flag of the one tile that has slots past kv_len, so that the others carry no masking code)
    // (par: compile-time parity of t - t0, which picks the stages: their offsets are then immediates of the LDS reads)
    auto tile_step = [&](auto tail_c, auto par_c, f32x16 (&s_cur)[2], f32x16 (&s_nxt)[2], int t) {
        constexpr bool tail = decltype(tail_c)::value;
        constexpr int rel = decltype(par_c)::value;
        wait_loads();
        barrier();                       // K(t+1) and V(t) have landed; everyone is done with K(t), V(t-1)
        if (tail) {
            blank_v_tail(t, rel & 1);
            __syncthreads();
        }
        const unsigned char* sk = k_stage + ((rel + 1) & 1) * K_TILE_BYTES;
        const unsigned char* sv = v_stage + (rel & 1) * V_TILE_BYTES;

        if (tail) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (t * KT + kb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3) >= kv_len) s_cur[kb][r] = -INFINITY;
        }
        // ---- S^T(t+1) on the matrix unit in two halves | under each, p = 2^(s c - m_run) of one 32-key block of
        // tile t on the vector unit, its row sum and its bf16 fragments.  m_run is the exponents' reference point, not
        // the exact running maximum: no maximum is formed here at all.  If a score has run more than about
        // log2(kSumLimit) ahead of it (or no key has been seen yet: m_run = -inf makes p infinite), this lane's sum of
        // p leaves the range, and the wave then takes the slow path below, which moves the reference point to the
        // true maximum, rescales the accumulators and forms p again.  The reference cancels in O / l.
        // (Past the last tile the matrix unit reads a stale stage and the result is dropped: no branch, so that matrix
        // and vector instructions share a basic block and can be interleaved.)
        // The loads of K(t+2) and V(t+1) go out between the first MFMAs, one each: issued in a burst after the barrier they
        // hold every wave of the unit (an issuing wave waits while the LDS pipeline takes in the loads before its own,
        // about 25 clocks each) with the matrix pipe idle.  They are unconditional: past the last tile they fetch it
        // again into a stage that nobody reads, so that matrix, vector and load instructions share a basic block.
        float ls[4];
        bf16x8 pf[4];
        auto exps = [&](int kb) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[kb][r], scale_log2e, -m_run));
                ls[r & 3] = (kb == 0 && r < 4) ? p : ls[r & 3] + p;     // four independent chains
                pf[kb * 2 + (r >> 3)][r & 7] = (bf16)p;
            }
        };
        __builtin_amdgcn_sched_barrier(0);
        qk_half(s_nxt, sk, 0, [&]() {
            load_k(min(t + 2, t1 - 1), rel & 1);
            load_v(min(t + 1, t1 - 1), (rel + 1) & 1);
        });
        exps(0);
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);       // the eight fragment reads, then MFMA | load | vector work
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (m < 2 * LPT) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        qk_half(s_nxt, sk, 1, nothing);
        exps(1);
        float lsum = (ls[0] + ls[1]) + (ls[2] + ls[3]);
        pin_fragments(pf);               // the bf16 fragments are formed here, among the MFMAs, not after the branch
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(lsum <= kSumLimit)) != 0, 0)) {
            // Slow path: move the reference point to the true row maximum (four independent chains; the same for the
            // two lanes of a query), rescale the accumulators and form p again.
            float mc[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                mc[c] = max3_f32(s_cur[0][4 * c], s_cur[1][4 * c], s_cur[0][4 * c + 1]);
                mc[c] = max3_f32(mc[c], s_cur[1][4 * c + 1], s_cur[0][4 * c + 2]);
                mc[c] = max3_f32(mc[c], s_cur[1][4 * c + 2], s_cur[0][4 * c + 3]);
                mc[c] = max2_f32(mc[c], s_cur[1][4 * c + 3]);
            }
            const float mx = max_xor32(max2_f32(max3_f32(mc[0], mc[1], mc[2]), mc[3]));
            const float m_new = fmaxf(m_run, mx * scale_log2e);     // finite: every tile has a valid key
            const bool moved = m_new > m_run + kMaxSlack;            // a query within kMaxSlack of its reference keeps it
            const float alpha = moved ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.0f;
            l_run *= alpha;
#pragma unroll
            for (int i = 0; i < D / 32; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) o_acc[i][r] *= alpha;
            m_run = moved ? m_new : m_run;
            exps(0);
            exps(1);
            lsum = (ls[0] + ls[1]) + (ls[2] + ls[3]);
            pin_fragments(pf);
        }
        l_run += lsum;
        __builtin_amdgcn_sched_barrier(0);

        // ---- O^T += V^T P^T : four steps of 16 keys; step ts uses registers 8 (ts % 2) .. + 7 of block ts / 2,
        // i.e. slots 16 ts + 4 (lane / 32) + {0..3} and 16 ts + 8 + 4 (lane / 32) + {0..3}: chunk 2 ts + lane / 32
        // of the V^T row in the cache's column order.
#pragma unroll
        for (int ts = 0; ts < 4; ++ts) {
#pragma unroll
            for (int db = 0; db < D / 32; ++db) {
                const unsigned char* vrow = sv + (db * 32 + l31) * 128;
                const bf16x8 vf = *reinterpret_cast<const bf16x8*>(vrow + (((2 * ts + lh) ^ ((l31 >> 1) & 7)) << 4));
                o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[ts], o_acc[db], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);       // fragment reads run six ahead of the MFMAs
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    if (t0 < t1) {
        // The wait counts loads: the queries and the first K tile are there when no more are in flight than went out behind
        // them.  So their order is held here.
        __builtin_amdgcn_sched_barrier(kNoMemory);
        load_k(t0, 0);
        __builtin_amdgcn_sched_barrier(kNoMemory);
        load_v(t0, 0);
        if (NW == 8) load_k(min(t0 + 1, t1 - 1), 1);
        __builtin_amdgcn_sched_barrier(kNoMemory);
        __builtin_amdgcn_s_waitcnt(0x0F70 | ((NW == 8 ? 2 : 1) * LPT));
        barrier();
        if (STAGED) read_queries(qf, q_stage, l31, lh);
        if (NW == 4) {
            if (STAGED) {                                    // everyone has its queries: the second K stage is free
                __builtin_amdgcn_s_waitcnt(0xC07F);
                barrier();
            }
            load_k(min(t0 + 1, t1 - 1), 1);
        }
        qk_half(s_a, k_stage, 0, nothing);
        qk_half(s_a, k_stage, 1, nothing);
        scale_log2e = query_scale(a, softmax_scale, row_of(query_in_chunk()), lh);
        if (zero_queries(qf, scale_log2e, softmax_scale)) {
            qk_half(s_a, k_stage, 0, nothing);
            qk_half(s_a, k_stage, 1, nothing);
        }
    }
    // full tiles in pairs (the two S^T register sets trade places), then what is left: at most one full tile
    // and the tail tile
    const std::false_type no_tail;
    const std::true_type with_tail;
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    int t = t0;
    for (; t + 2 <= t_full; t += 2) {
        tile_step(no_tail, even, s_a, s_b, t);
        tile_step(no_tail, odd, s_b, s_a, t + 1);
    }
    if (t < t_full) {
        tile_step(no_tail, even, s_a, s_b, t);
        if (t_full < t1) tile_step(with_tail, odd, s_b, s_a, t_full);
    } else if (t_full < t1) {
        tile_step(with_tail, even, s_a, s_b, t_full);
    }

    // ---- finish: divide by the row sum and write (no direct load may still be on its way to this LDS when the wave ends)
    wait_loads();
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    const float inv_l = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    const int q_in_chunk = query_in_chunk();
    const size_t q_row = row_of(q_in_chunk);
    if (a.splits == 1) {
        bf16* op = a.o + q_row * C + h * D + 8 * lh;
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
                bf16x4 w[2];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    w[0][e] = (bf16)(o_acc[db][4 * g + e] * inv_l);
                    w[1][e] = (bf16)(o_acc[db][4 * g + 4 + e] * inv_l);
                }
                const uint4 v = eight_channels(w[0], w[1]);
                if (q_in_chunk < a.L) *reinterpret_cast<uint4*>(op + db * 32 + 8 * g) = v;
            }
        }
    } else if (q_in_chunk < a.L) {
        const size_t rows = (size_t)a.B * a.L;
        float* op = a.part_o + ((size_t)split * rows + q_row) * C + h * D + 4 * lh;
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = o_acc[db][4 * g + e] * inv_l;
                *reinterpret_cast<f32x4*>(op + db * 32 + 8 * g) = w;
            }
        }
        if (own_lane() < 32) {
            float* ml = a.part_ml + (((size_t)split * rows + q_row) * a.H + h) * 2;
            ml[0] = m_run;
            ml[1] = l_tot;
        }
    }
}

template <int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void attention_kernel(AttnArgs a, float softmax_scale) {
    attention_body<NW, true>(a, softmax_scale);
}
template <int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void attention_any_address_kernel(AttnArgs a, float softmax_scale) {
    attention_body<NW, false>(a, softmax_scale);
}

// With workgroups behind its own that fetch memory; kernels of their own, because in the same ones the few instructions more
// cost every launch 0.4 us a round.
template <int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void attention_fetching_kernel(AttnArgs a, float softmax_scale, WarmArgs warm) {
    if (blockIdx.x >= a.n_wg) return warm_memory(warm, blockIdx.x - a.n_wg);
    attention_body<NW, true>(a, softmax_scale);
}

// ---------------------------------------------------------------------------------------------------
// Key-split form for skinny launches (a single 1024-token chunk: heads x query tiles is well below the number of
// SIMDs).  A workgroup is NQ query blocks x NKW key slices = 8 waves: it walks the whole key range in tiles of
// 32 NKW keys, wave (qb, kw) computing the scores of its 32 queries against keys 32 kw .. 32 kw + 31 of every tile
// and keeping its own running maximum, sum and output; at the end the NKW partial results of a query block are
// merged through LDS.  Compared with splitting the key range over workgroups this needs no partial outputs in
// memory and no merge kernel, and every K / V^T tile staged in LDS still serves all eight waves.
//   K stage:   32 NKW keys x 256 B, chunk c of row r at position c ^ (r % 16)
//   V^T stage: 128 rows (d) x 32 NKW keys (64 NKW bytes; 256 B for NKW = 4), same swizzle
// Needs cap % (32 NKW) == 0 (a tile never reaches past a V^T row).
template <int NQ, int NKW, bool STAGED>
__device__ __forceinline__ void attention_ks_body(const AttnArgs& a, float softmax_scale) {
    static_assert(NKW == 4 && NQ * NKW == 8, "tiles of 128 keys, eight waves");
    constexpr int NW = NQ * NKW;
    constexpr int QT = 32 * NQ;
    constexpr int KTT = 32 * NKW;                         // keys per tile
    constexpr int ROWB = 256;                             // bytes per LDS row of either stage
    constexpr int K_BYTES = KTT * ROWB;                   // 32 KB
    constexpr int V_BYTES = D * ROWB;                     // 32 KB
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    unsigned char* const k_stage = smem_raw;                          // [2][K_BYTES]
    unsigned char* const v_stage = smem_raw + 2 * K_BYTES;            // [2][V_BYTES]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qb = wave % NQ;
    const int kw = wave / NQ;
    const int l31 = lane & 31;
    const int lh = lane >> 5;

    int qt, h, b;
    locate(a, qt, h, b);
    const int C = a.H * D;

    const StreamKeys keys = stream_keys(a, b);
    const int cap = keys.cap, kv_len = keys.kv_len;
    const int n_tiles = (int)((unsigned)(kv_len + KTT - 1) / KTT);    // one at least
    const int tail_tile = (kv_len % KTT) ? n_tiles - 1 : -1;

    const int q_in_chunk = qt * QT + qb * 32 + l31;
    const size_t q_row = (size_t)(unsigned)b * (unsigned)a.L + (unsigned)min(q_in_chunk, a.L - 1);
    // the workgroup's 64 queries go through the second V^T stage, which is free until the first tile is done: two loads per wave
    unsigned char* const q_stage = v_stage + V_BYTES;
    bf16x8 qf[D / 16];
    if (STAGED) load_queries<2>(a, b, h, qt * QT, wave * 8, lane, q_stage, C);
    else fetch_queries(qf, a, q_row, h, lh, C);

    // A wave load fills four 256-byte rows; wave w issues loads w, w + 8, w + 16, w + 24 of each tile.
    const unsigned char* kbase = reinterpret_cast<const unsigned char*>(keys.k + (size_t)h * cap * D);
    const unsigned char* vbase = reinterpret_cast<const unsigned char*>(keys.vt + (size_t)h * D * cap);
    constexpr int LPT = KTT / 4 / NW;                     // 4 wave loads per tile and operand for each wave
    const int ld_row = 4 * wave + (lane >> 4);                                    // + 32 i
    const int ld_chunk = (lane & 15) ^ (ld_row & 15);                             // 32 i does not change row % 16
    const uint32_t k_off = (uint32_t)ld_row * ROWB + (uint32_t)ld_chunk * 16;
    const size_t v_off = (size_t)ld_row * cap * 2 + (size_t)ld_chunk * 16;
    // (a tile index past the last tile fetches the last tile again, into a stage that nobody reads any more: the loads
    // are unconditional so that they can sit among the matrix instructions of a basic block)
    auto load_k = [&](int t, int stage) {
        const unsigned char* src = kbase + (size_t)min(t, n_tiles - 1) * K_BYTES + k_off;
        unsigned char* dst = k_stage + stage * K_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < LPT; ++i) load_to_lds_b128(src + i * (NW * 1024), dst + i * (NW * 1024));
    };
    auto load_v = [&](int t, int stage) {
        const unsigned char* src = vbase + (size_t)min(t, n_tiles - 1) * (KTT * 2) + v_off;
        unsigned char* dst = v_stage + stage * V_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < LPT; ++i) load_to_lds_b128(src + (size_t)i * 32 * cap * 2, dst + i * (NW * 1024));
    };
    // Slots past kv_len may hold anything (NaN included) and 0 x NaN is not 0: blank them in the staged V^T tile.
    auto blank_v_tail = [&](int t, int stage) {
        const int n_valid = kv_len - t * KTT;
        bf16* sv = reinterpret_cast<bf16*>(v_stage + stage * V_BYTES);
        for (int idx = tid; idx < D * 16; idx += 64 * NW) {
            const int row = idx >> 4, p = idx & 15;
            const int c = p ^ (row & 15);
            bf16x8 v = *reinterpret_cast<bf16x8*>(sv + row * (ROWB / 2) + p * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int u = 8 * c + e;                                          // stored column
                const int slot = (u & ~12) | ((u & 4) << 1) | ((u & 8) >> 1);     // slot it holds
                if (slot >= n_valid) v[e] = (bf16)0.0f;
            }
            *reinterpret_cast<bf16x8*>(sv + row * (ROWB / 2) + p * 8) = v;
        }
    };

    f32x16 o_acc[D / 32];
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o_acc[i][r] = 0.0f;
    float m_run = kNoKey;        // finite: a fully masked slice has scores of -inf, and -inf + inf is not a number
    float l_run = 0.0f;

    // Half of S^T of this wave's 32 keys of the tile in stage sk: d steps 4 half .. 4 half + 3.
    // this lane's eight K fragments and its two V^T fragments of a step in the first 32-row block, all in stage 0: the
    // stage and the block add compile-time constants, which the LDS reads take as immediates
    const unsigned char* kfrag[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; ++i) kfrag[i] = k_stage + (kw * 32 + l31) * ROWB + (((2 * i + lh) ^ (l31 & 15)) << 4);
    const unsigned char* vfrag[2];
#pragma unroll
    for (int ts = 0; ts < 2; ++ts) vfrag[ts] = v_stage + l31 * ROWB + (((4 * kw + 2 * ts + lh) ^ (l31 & 15)) << 4);
    auto qk_half = [&](f32x16& s, int stage, int half, auto&& after_reads) {
        if (half == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.0f;
        }
        bf16x8 kf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            kf[i] = *reinterpret_cast<const bf16x8*>(kfrag[4 * half + i] + stage * K_BYTES);
        after_reads();
#pragma unroll
        for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[4 * half + i], s, 0, 0, 0);
    };
    auto nothing = []() {};
    auto wait_loads = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); };       // vmcnt(0) only
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    float scale_log2e = softmax_scale;
    f32x16 s_a, s_b;
    auto tile_step = [&](auto tail_c, auto par_c, f32x16& s_cur, f32x16& s_nxt, int t) {
        constexpr bool tail = decltype(tail_c)::value;
        constexpr int par = decltype(par_c)::value;      // parity of t, at compile time: stage offsets become immediates
        wait_loads();
        barrier();                       // K(t+1) and V(t) have landed; everyone is done with K(t), V(t-1)
        if (tail) {
            blank_v_tail(t, par);
            __syncthreads();
        }
        constexpr int sk = par ^ 1;          // stage of K(t+1)
        if (tail) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (t * KTT + kw * 32 + 8 * (r >> 2) + 4 * lh + (r & 3) >= kv_len) s_cur[r] = -INFINITY;
        }
        // ---- S^T(t+1) on the matrix unit in two halves | p of tile t on the vector unit, without a row maximum
        // (see attention_kernel): the slow path is taken when a sum of p has left the range, which is also what
        // happens at a lane's first valid key (m_run = kNoKey: p infinite).  A lane whose slice lies past kv_len has
        // scores of -inf, p = 0 and keeps kNoKey (finite, so that -inf - m_run is not "not a number").
        float ls[4];
        bf16x8 pf[2];
        auto exps = [&](int h) {
#pragma unroll
            for (int r = 8 * h; r < 8 * h + 8; ++r) {
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[r], scale_log2e, -m_run));
                ls[r & 3] = r < 4 ? p : ls[r & 3] + p;
                pf[r >> 3][r & 7] = (bf16)p;
            }
        };
        __builtin_amdgcn_sched_barrier(0);
        // the loads of K(t+2) go out between the MFMAs of the first half, those of V(t+1) between those of the second
        qk_half(s_nxt, sk, 0, [&]() { load_k(t + 2, par); });
        exps(0);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        qk_half(s_nxt, sk, 1, [&]() { load_v(t + 1, par ^ 1); });
        exps(1);
        float lsum = (ls[0] + ls[1]) + (ls[2] + ls[3]);
        pin_fragments(pf);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(lsum <= kSumLimit)) != 0, 0)) {
            float mc[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) mc[c] = max2_f32(max3_f32(s_cur[4 * c], s_cur[4 * c + 1], s_cur[4 * c + 2]), s_cur[4 * c + 3]);
            const float mx = max_xor32(max2_f32(max3_f32(mc[0], mc[1], mc[2]), mc[3]));
            const float m_new = fmaxf(m_run, mx * scale_log2e);       // stays kNoKey in a lane that has still seen no key
            const bool moved = m_new > m_run + kMaxSlack;
            const float al = moved ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.0f;
            l_run *= al;
#pragma unroll
            for (int i = 0; i < D / 32; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) o_acc[i][r] *= al;
            m_run = moved ? m_new : m_run;
            exps(0);
            exps(1);
            lsum = (ls[0] + ls[1]) + (ls[2] + ls[3]);
            pin_fragments(pf);
        }
        l_run += lsum;
        __builtin_amdgcn_sched_barrier(0);
        // ---- O^T += V^T P^T: two steps of 16 keys; chunk 4 kw + 2 ts + lh of the V^T row in the cache's column order
#pragma unroll
        for (int ts = 0; ts < 2; ++ts) {
#pragma unroll
            for (int db = 0; db < D / 32; ++db) {
                const bf16x8 vf = *reinterpret_cast<const bf16x8*>(vfrag[ts] + par * V_BYTES + db * 32 * ROWB);
                o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[ts], o_acc[db], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // in this order (see attention_body): the wait counts what went out behind the queries and the first K tile
    __builtin_amdgcn_sched_barrier(kNoMemory);
    load_k(0, 0);
    __builtin_amdgcn_sched_barrier(kNoMemory);
    load_v(0, 0);
    load_k(1, 1);
    __builtin_amdgcn_sched_barrier(kNoMemory);
    __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * LPT));
    barrier();
    if (STAGED) read_queries(qf, q_stage + qb * 8192, l31, lh);
    qk_half(s_a, 0, 0, nothing);
    qk_half(s_a, 0, 1, nothing);
    scale_log2e = query_scale(a, softmax_scale, q_row, lh);
    if (zero_queries(qf, scale_log2e, softmax_scale)) {
        qk_half(s_a, 0, 0, nothing);
        qk_half(s_a, 0, 1, nothing);
    }
    const int t_full = (tail_tile >= 0) ? n_tiles - 1 : n_tiles;        // tiles [0, t_full) have 128 valid slots
    const std::false_type no_tail;
    const std::true_type with_tail;
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    int t = 0;
    for (; t + 2 <= t_full; t += 2) {
        tile_step(no_tail, even, s_a, s_b, t);
        tile_step(no_tail, odd, s_b, s_a, t + 1);
    }
    if (t < t_full) {
        tile_step(no_tail, even, s_a, s_b, t);
        if (t_full < n_tiles) tile_step(with_tail, odd, s_b, s_a, t_full);
    } else if (t_full < n_tiles) {
        tile_step(with_tail, even, s_a, s_b, t_full);
    }

    // ---- merge the NKW partial results of each query block through LDS (the stages are free once every wave is past the
    // first barrier; the sums and reference points lie behind them).  A wave writes the channels that the others add up and
    // keeps its own 32: the writes are what this costs (13 clocks per KB).
    wait_loads();                                         // nor may a tile fetched past the end still be on its way to them
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    float* const xm = reinterpret_cast<float*>(smem_raw + 4 * K_BYTES);           // [NW][32] maxima, after the stages
    float* const xl = xm + NW * 32;                                               // [NW][32] sums
    f32x4* const ox = reinterpret_cast<f32x4*>(smem_raw);                         // [NW][4 db][4][64] weighted outputs
    if (lh == 0) {
        xm[wave * 32 + l31] = m_run;
        xl[wave * 32 + l31] = l_tot;
    }
    __syncthreads();
    // a slice that saw no key has m = kNoKey and l = 0: weight 2^(kNoKey - mmax) = 0, or 1 times l = 0 if all are such
    float mmax = kNoKey;
#pragma unroll
    for (int k = 0; k < NKW; ++k) mmax = fmaxf(mmax, xm[(qb + NQ * k) * 32 + l31]);
    float lsum = 0.0f;
#pragma unroll
    for (int k = 0; k < NKW; ++k)
        lsum += xl[(qb + NQ * k) * 32 + l31] * __builtin_amdgcn_exp2f(xm[(qb + NQ * k) * 32 + l31] - mmax);
    const float wgt = lsum > 0.0f ? __builtin_amdgcn_exp2f(m_run - mmax) / lsum : 0.0f;
    f32x4 own[4];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = o_acc[db][4 * g + e] * wgt;
            if (db == kw) own[g] = v;
            else ox[((wave * 4 + db) * 4 + g) * 64 + lane] = v;
        }
    }
    __syncthreads();
    // wave (qb, kw) adds up, in the order of the slices, and writes the 32 channels db = kw of its query block
    bf16* op = a.o + q_row * C + h * D + kw * 32 + 8 * lh;
#pragma unroll
    for (int g = 0; g < 4; g += 2) {
        bf16x4 w[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < NKW; ++k) acc += k == kw ? own[g + i] : ox[(((qb + NQ * k) * 4 + kw) * 4 + g + i) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[i][e] = (bf16)acc[e];
        }
        const uint4 v = eight_channels(w[0], w[1]);
        if (q_in_chunk < a.L) *reinterpret_cast<uint4*>(op + 8 * g) = v;
    }
}

template <int NQ, int NKW>
__global__ __launch_bounds__(64 * NQ * NKW, 1) void attention_ks_kernel(AttnArgs a, float softmax_scale) {
    attention_ks_body<NQ, NKW, true>(a, softmax_scale);
}
template <int NQ, int NKW>
__global__ __launch_bounds__(64 * NQ * NKW, 1) void attention_ks_any_address_kernel(AttnArgs a, float softmax_scale) {
    attention_ks_body<NQ, NKW, false>(a, softmax_scale);
}

template <int NQ, int NKW>
__global__ __launch_bounds__(64 * NQ * NKW, 1) void attention_ks_fetching_kernel(AttnArgs a, float softmax_scale, WarmArgs warm) {
    if (blockIdx.x >= a.n_wg) return warm_memory(warm, blockIdx.x - a.n_wg);
    attention_ks_body<NQ, NKW, true>(a, softmax_scale);
}

// out = sum_i w_i O_i / sum_i w_i,  w_i = l_i 2^(m_i - max m).  One thread per four channels.
__global__ __launch_bounds__(256) void attention_merge_kernel(AttnArgs a) {
    const int C = a.H * D;
    const size_t rows = (size_t)a.B * a.L;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;     // over rows * C / 4
    if (idx >= rows * (C / 4)) return;
    const size_t row = idx / (C / 4);
    const int c4 = (int)(idx - row * (C / 4)) * 4;
    const int h = c4 / D;
    float m[16], l[16];
    float mmax = -INFINITY;
    for (int s = 0; s < a.splits; ++s) {
        const float* ml = a.part_ml + (((size_t)s * rows + row) * a.H + h) * 2;
        m[s] = ml[0];
        l[s] = ml[1];
        mmax = fmaxf(mmax, m[s]);
    }
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    float wsum = 0.0f;
    for (int s = 0; s < a.splits; ++s) {
        const float w = l[s] > 0.0f ? l[s] * __builtin_amdgcn_exp2f(m[s] - mmax) : 0.0f;
        const f32x4 o = *reinterpret_cast<const f32x4*>(a.part_o + ((size_t)s * rows + row) * C + c4);
        acc += o * w;
        wsum += w;
    }
    const float inv = 1.0f / wsum;
    bf16x4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = (bf16)(acc[e] * inv);
    *reinterpret_cast<bf16x4*>(a.o + row * C + c4) = out;
}

}  // namespace

// Waves per workgroup: 4 (128 queries, two workgroups per compute unit) or 8 (256 queries, one workgroup per unit,
// half the K/V traffic from the L2 per query).
// Overrides for tuning runs and tests, set through sdv2_tuning_set("attn_waves" / "attn_splits", ...); 0 = the plan's
// own choice.  attn_waves 4 / 8: that many query blocks per workgroup, one key stream; 2: the key-split form.
static int g_force_waves = 0;
static int g_force_splits = 0;
void set_attention_overrides(int waves, int splits) {
    if (waves >= 0) g_force_waves = (waves == 4 || waves == 8 || waves == 2) ? waves : 0;
    if (splits >= 0) g_force_splits = splits > 16 ? 16 : splits;
}

// Forms of a launch: workgroups of 4 waves (128 queries, two workgroups per compute unit) or 8 waves (256 queries, one per unit,
// half the K/V traffic from the L2 per query), each with the key range whole or in parts (most_parts) that a merge pass joins; and the key-split form (2 query blocks x 4 key slices, one workgroup per unit), for capacities of whole 128-key
// tiles.  Microseconds of a launch:  c + rounds (tiles a + b), rounds as for the tiles of a product (a workgroup per slot is a
// round; of a last round that fills the share x of the slots the part p + s x, two per unit beyond a half q + (1 - q) x), and
// m + n per MB that the merge reads and writes.  Fitted to 2616 launches (4 to 40 heads, 16 to 12 480 keys, 1 to 8 streams, keys
// and values cold): rms error 4, 4 and 7 %.  On 1308 others the form picked is on average 0.3 % slower than the best of all;
// the thresholds that this replaces, workgroups against units alone, 9 %: 1560 x 12 heads over 512 keys 18.2 -> 12.9 us, over
// 4680 keys 93.8 -> 63.3, 8 x 1024 x 12 heads over 3072 keys 158.7 -> 148.9, 640 x 5 heads over 5120 keys 41.1 -> 27.9.
struct FormCost {
    int waves, queries, keys, slots;
    float a, b, c, p, s, q, m, n;
};
const FormCost kForms[] = {{4, 128, 64, 2 * kUnits, 1.768f, 6.58f, 2.82f, 0.453f, 0.265f, 0.658f, 5.25f, 0.104f},
                           {8, 256, 64, kUnits, 1.596f, 8.00f, 0.96f, 0.743f, 0.257f, 0.0f, 6.24f, 0.096f},
                           {2, 64, 128, kUnits, 1.134f, 5.17f, 2.05f, 0.763f, 0.237f, 0.0f, 0.0f, 0.0f}};
static const FormCost& form_of(int waves) { return kForms[waves == 2 ? 2 : waves == 8 ? 1 : 0]; }
constexpr int kMostParts = 16, kLeastTiles = 6;
constexpr float kPartsMargin = 1.03f;     // a split has to be that much better by the estimate: it needs scratch and a second launch

static float attention_cost(const FormCost& f, int B, int L, int H, int max_kv, int parts) {
    const long long wgs = (long long)((L + f.queries - 1) / f.queries) * H * B * parts;
    const int tiles = ((max_kv + f.keys - 1) / f.keys + parts - 1) / parts;
    const float full = (float)(wgs / f.slots), x = (float)(wgs % f.slots) / (float)f.slots;
    float last = 0.0f;
    if (x > 0.0f) last = f.slots == kUnits || x <= 0.5f ? f.p + f.s * x : f.q + (1.0f - f.q) * x;
    float us = f.c + (full + last) * ((float)tiles * f.a + f.b);
    if (parts > 1) us = (us + f.m + f.n * 1e-6f * (float)B * L * H * D * (8.0f * parts + 2.0f)) * kPartsMargin;
    return us;
}

// The most parts that a launch makes, for which its workspace has room: no more workgroups than have a place at once, at least
// six tiles each.  It never falls with more keys, as the best number of parts may (748 x 9 heads: nine over 7003 keys, eight over
// 8648), so a workspace for the longest key range serves every shorter one.  The places are those of the 256-query form where its
// workgroups give at least half of the units one, of the 128-query form elsewhere; either way parts x queries x heads stay within
// 65 536.  Of 3924 measured launches two would take more parts, and gain nothing by them.
static int most_parts(int B, int L, int H, int max_kv) {
    const int tiles = (max_kv + KT - 1) / KT;
    if (g_force_splits > 0) {
        int n = g_force_splits;
        while (n > 1 && tiles / n < 2) --n;
        return n;
    }
    const bool wide = g_force_waves == 8 || (g_force_waves != 4 && (long long)((L + 255) / 256) * H * B >= kUnits / 2);
    const FormCost& form = form_of(wide ? 8 : 4);
    const long long wgs = (long long)((L + form.queries - 1) / form.queries) * H * B;
    if (wgs >= form.slots / 2) return 1;
    const int by_slots = (int)(form.slots / wgs), by_tiles = tiles / kLeastTiles;
    const int n = by_slots < by_tiles ? by_slots : by_tiles;
    return n < 1 ? 1 : n > kMostParts ? kMostParts : n;
}

struct AttnPlan {
    int waves, splits;      // of kForms
    float us;               // its estimate
};
// At most 33 estimates (0.1 to 0.3 us), formed anew for each launch.
static AttnPlan attention_plan(int B, int L, int H, int max_kv, bool key_split) {
    AttnPlan best{4, 1, 1e30f};
    const int most = most_parts(B, L, H, max_kv);
    for (int f = 0; f < 2; ++f) {
        const FormCost& form = kForms[f];
        if (key_split && g_force_waves == 2) break;
        if ((g_force_waves == 4 || g_force_waves == 8) && form.waves != g_force_waves) continue;
        for (int parts = g_force_splits > 0 ? most : 1; parts <= most; ++parts) {
            const float us = attention_cost(form, B, L, H, max_kv, parts);
            if (us < best.us) best = AttnPlan{form.waves, parts, us};
        }
    }
    if (key_split && (g_force_waves == 0 || g_force_waves == 2)) {
        const float us = attention_cost(form_of(2), B, L, H, max_kv, 1);
        if (us < best.us) best = AttnPlan{2, 1, us};
    }
    return best;
}

// While a cache fills, a launch goes by the keys that are there: with the form and parts of a full cache the first chunks took
// longer (a step of 1024 x 8 heads with room for 7168 keys, us a layer: first chunk 134.1 -> 120.9, second 137.1 -> 130.6; 20 heads,
// first chunk 294.3 -> 251.9).  But a recorded step has the full cache's, and other parts add in another order, so an eager one
// differs only where a tenth of the launch is to be had, more than the estimates are off by.
constexpr float kWorthAnotherForm = 1.1f;

void plan_attention(AttnLaunch* a) {
    int max_kv = 0;
    bool key_split = true;
    for (int b = 0; b < a->B; ++b) {
        if (a->cap[b] % 128) key_split = false;
        max_kv = a->kv_len[b] > max_kv ? a->kv_len[b] : max_kv;
    }
    AttnPlan p = attention_plan(a->B, a->L, a->H, max_kv, key_split);
    if (a->full_kv > max_kv) {
        const AttnPlan full = attention_plan(a->B, a->L, a->H, a->full_kv, key_split);
        const float us = attention_cost(form_of(full.waves), a->B, a->L, a->H, max_kv, full.splits);
        if (us <= kWorthAnotherForm * p.us) p = AttnPlan{full.waves, full.splits, us};
    }
    a->waves = p.waves;
    a->splits = p.splits;
    a->us = p.us;
}

size_t attention_workspace_bytes(int B, int L, int C, int max_kv_len) {
    const int H = C / D;
    const int splits = most_parts(B, L, H, max_kv_len);
    if (splits == 1) return 0;
    const size_t rows = (size_t)B * L;
    return (size_t)splits * rows * C * sizeof(float) + (size_t)splits * rows * H * 2 * sizeof(float);
}

// most_parts at its most: 16 parts, at least six key tiles each, parts * B * L * H up to 65 536.
size_t attention_workspace_bytes_bound(int B, int L, int C, int max_kv_len) {
    const size_t H = C / D, most_rows = 512 * 128 / H;
    const int by_tiles = (max_kv_len + KT - 1) / KT / 6;
    const size_t parts = by_tiles < 16 ? by_tiles : 16;
    const size_t rows = parts * B * L < most_rows ? parts * B * L : most_rows;
    const size_t bound = parts <= 1 ? 0 : rows * (C * sizeof(float) + H * 2 * sizeof(float));
    const size_t planned = attention_workspace_bytes(B, L, C, max_kv_len);      // above the bound only for a forced number of parts
    return planned > bound ? planned : bound;
}

static void kernel_name(char* out, size_t cap, int waves, const char* variant) {
    if (waves == 2) snprintf(out, cap, "attention_ks_%skernel<2, 4>", variant);
    else snprintf(out, cap, "attention_%skernel<%d>", variant, waves);
}

void attention_plan_name(const AttnLaunch& a, char* out, size_t cap) { kernel_name(out, cap, a.waves, ""); }

// Direct loads of the queries go from memory to LDS in pieces of 16 bytes, which have to start at multiples of 16 (rows and
// heads are multiples of 256 bytes, so the first address decides); queries at any other address of a bf16 are fetched into registers.
static bool queries_aligned(const AttnArgs& a) { return (reinterpret_cast<uintptr_t>(a.q) & 15) == 0; }

IdleUnits attention_idle_units(const AttnLaunch& a) {
    const FormCost& f = form_of(a.waves);
    const int wgs = (a.L + f.queries - 1) / f.queries * a.H * a.B * a.splits;
    IdleUnits idle{0, f.waves == 4 ? 4u : 8u, a.us};
    if (wgs < kUnits) idle.blocks = (unsigned)(kUnits - wgs);
    return idle;
}

hipError_t launch_attention(const AttnLaunch& launch, hipStream_t s, int part, const WarmArgs* side) {
    AttnArgs a = launch;
    const int waves = launch.waves;
    auto one_dimension = [&](int q_tiles, int parts) {
        a.n_wg = (unsigned)q_tiles * a.H * a.B * parts;
        a.by_q_tiles = fast_div(q_tiles, a.n_wg);
        a.by_heads = fast_div(a.H, a.n_wg);
        return dim3(a.n_wg);
    };
    constexpr size_t smem = (size_t)2 * K_TILE_BYTES + 2 * V_TILE_BYTES, smem8 = smem + 8 * 8192;      // eight waves: their queries behind the stages
    constexpr size_t smem_ks = (size_t)4 * 32768 + 2 * 8 * 32 * sizeof(float);     // four 32 KB stages + the (m, l) exchange
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    typedef void (*Kernel)(AttnArgs, float);
    typedef void (*FetchingKernel)(AttnArgs, float, WarmArgs);
    std::call_once(attr_once, [&]() {
        const std::pair<Kernel, size_t> kernels[] = {{attention_kernel<4>, smem},
                                                     {attention_kernel<8>, smem8},
                                                     {attention_ks_kernel<2, 4>, smem_ks},
                                                     {attention_any_address_kernel<4>, smem},
                                                     {attention_any_address_kernel<8>, smem8},
                                                     {attention_ks_any_address_kernel<2, 4>, smem_ks}};
        for (const auto& k : kernels)
            if (attr_err == hipSuccess)
                attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(k.first), hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.second);
        const std::pair<FetchingKernel, size_t> fetching[] = {
            {attention_fetching_kernel<4>, smem}, {attention_fetching_kernel<8>, smem8}, {attention_ks_fetching_kernel<2, 4>, smem_ks}};
        for (const auto& k : fetching)
            if (attr_err == hipSuccess)
                attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(k.first), hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.second);
    });
    if (attr_err != hipSuccess || attributes_only()) return attr_err;
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)D);
    const bool staged = queries_aligned(a), fetching = side != nullptr && side->blocks > 0 && staged;
    if (g_launch_note.on && part != 2)
        kernel_name(g_launch_note.kernel, sizeof(g_launch_note.kernel), waves, fetching ? "fetching_" : staged ? "" : "any_address_");
    if (waves == 2) {
        if (part == 2) return hipSuccess;
        const dim3 grid = one_dimension((a.L + 63) / 64, 1);
        const Kernel kernel = staged ? attention_ks_kernel<2, 4> : attention_ks_any_address_kernel<2, 4>;
        if (fetching) hipLaunchKernelGGL((attention_ks_fetching_kernel<2, 4>), dim3(grid.x + side->blocks), dim3(512), smem_ks, s, a, scale_log2e, *side);
        else hipLaunchKernelGGL(kernel, grid, dim3(512), smem_ks, s, a, scale_log2e);
        return hipGetLastError();
    }
    hipError_t e = hipSuccess;
    if (part != 2) {
        const int queries = 32 * waves;
        const dim3 grid = one_dimension((a.L + queries - 1) / queries, a.splits);
        if (fetching && waves == 8)
            hipLaunchKernelGGL(attention_fetching_kernel<8>, dim3(grid.x + side->blocks), dim3(512), smem8, s, a, scale_log2e, *side);
        else if (fetching)
            hipLaunchKernelGGL(attention_fetching_kernel<4>, dim3(grid.x + side->blocks), dim3(256), smem, s, a, scale_log2e, *side);
        else if (waves == 8) hipLaunchKernelGGL(staged ? attention_kernel<8> : attention_any_address_kernel<8>, grid, dim3(512), smem8, s, a, scale_log2e);
        else hipLaunchKernelGGL(staged ? attention_kernel<4> : attention_any_address_kernel<4>, grid, dim3(256), smem, s, a, scale_log2e);
        e = hipGetLastError();
    }
    if (e != hipSuccess || part == 1) return e;
    if (a.splits > 1) {
        const size_t n = (size_t)a.B * a.L * (a.H * D / 4);
        hipLaunchKernelGGL(attention_merge_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace sdv2
