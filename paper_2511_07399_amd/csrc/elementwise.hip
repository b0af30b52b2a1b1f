// HBM-bound kernels of the block: LayerNorm with adaLN modulation, RMSNorm, the fused
// q/k RMSNorm + 3D-RoPE + rolling-cache append, cache re-layouts and the small conditioning GEMVs.
//
// These are the "36 b L_q C" activation bytes and the "4 b L_q C" cache write of the memory model
// in Appendix B of the paper.  The paper's implementation also pays for sliding-window buffering and
// concatenation (its measured extra traffic gamma); here a chunk's keys and values are written once,
// straight into their ring slots, and nothing is ever moved.
//
// Row reductions use cross-lane shuffles inside a wavefront (RMSNorm, the q/k norm: one wavefront per row;
// LayerNorm: two wavefronts per row that exchange their partial sums through LDS); no atomics.
#include "common.h"

namespace sdv2 {

namespace {

// ------------------------------------------------------------------ LayerNorm (+ modulation or affine)
// Two wavefronts per row, two rows per workgroup: a row of the small model is only 6 KB, and with one
// wavefront per row the kernel is a chain of latencies (load, two shuffle reductions, store) on a quarter of
// the chip's wave slots.  Mean and variance come from one pass over the registers, as sums of (x - x[0])
// and (x - x[0])^2 (shifting by the row's first element keeps the fp32 variance exact enough whatever the
// row's mean); the two waves of a row exchange their partial sums through LDS.
// LN_MAXV = float4 values a lane keeps in registers: C <= 512 * LN_MAXV.
// EARLY: scale and shift are fetched together with the row instead of after the reduction.  With few rows the kernel
// is a chain of latencies and theirs would come on top of the row's; with many rows it is bound by bandwidth and the
// extra registers would only cost occupancy.
template <int LN_MAXV, bool EARLY>
__global__ __launch_bounds__(256) void layernorm_kernel(LnArgs a) {
    __shared__ float part[2][2][2];                       // [row in workgroup][wave of the row][sum, sum of squares]
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int rw = wave >> 1;                             // row in the workgroup
    const int half = wave & 1;
    const int t = half * 64 + lane;                       // 0 .. 127 within the row
    const int row_raw = blockIdx.x * 2 + rw;
    const bool live = row_raw < a.rows;
    const int row = live ? row_raw : a.rows - 1;          // a spare half workgroup recomputes the last row, stores nothing
    const int nvec = a.C >> 2;
    const f32x4* xp = reinterpret_cast<const f32x4*>(a.x + (size_t)row * a.C);
    const float pivot = a.x[(size_t)row * a.C];
    f32x4 v[LN_MAXV];
    f32x4 sc[EARLY ? LN_MAXV : 1], sh[EARLY ? LN_MAXV : 1];
    const int stream = row / a.rows_per_stream;
    auto fetch_affine = [&](int c, f32x4& scv, f32x4& shv) {
        scv = *reinterpret_cast<const f32x4*>(a.scale_a + c);
        shv = *reinterpret_cast<const f32x4*>(a.shift_a + c);
        if (a.scale_b != nullptr) {
            scv += *reinterpret_cast<const f32x4*>(a.scale_b + (size_t)stream * a.b_stride + c);
            shv += *reinterpret_cast<const f32x4*>(a.shift_b + (size_t)stream * a.b_stride + c);
            scv += 1.0f;
        }
    };
    float sum = 0.0f, sq = 0.0f;
#pragma unroll
    for (int i = 0; i < LN_MAXV; ++i) {
        const int idx = t + 128 * i;
        if (idx < nvec) {
            v[i] = xp[idx];
            if (EARLY) fetch_affine(idx * 4, sc[i], sh[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < LN_MAXV; ++i) {
        const int idx = t + 128 * i;
        if (idx < nvec) {
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
        part[rw][half][0] = sum;
        part[rw][half][1] = sq;
    }
    __syncthreads();
    sum = part[rw][0][0] + part[rw][1][0];
    sq = part[rw][0][1] + part[rw][1][1];
    const float inv_c = 1.0f / (float)a.C;
    const float dmean = sum * inv_c;                      // mean - pivot
    const float var = fmaxf(sq * inv_c - dmean * dmean, 0.0f);
    const float rstd = rsqrtf(var + a.eps);
    const float mean = pivot + dmean;
    if (!live) return;
    bf16* op = a.out + (size_t)row * a.C;
#pragma unroll
    for (int i = 0; i < LN_MAXV; ++i) {
        const int idx = t + 128 * i;
        if (idx < nvec) {
            if (!EARLY) fetch_affine(idx * 4, sc[0], sh[0]);
            const f32x4 scv = sc[EARLY ? i : 0], shv = sh[EARLY ? i : 0];
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)((v[i][e] - mean) * rstd * scv[e] + shv[e]);
            *reinterpret_cast<bf16x4*>(op + idx * 4) = o;
        }
    }
}

// ------------------------------------------------------------------ RMSNorm in place on bf16 rows
// One wavefront per row; the row (NV 16-byte pieces per lane) and the gains are fetched once and stay in registers.
template <int NV>
__global__ __launch_bounds__(256) void rmsnorm_inplace_kernel(bf16* x, const float* gain, int rows, int C, int ld,
                                                              float eps) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    bf16* xp = x + (size_t)row * ld;
    const int nvec = C >> 3;
    bf16x8 v[NV];
    f32x4 g0[NV], g1[NV];
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + 64 * i;
        if (idx < nvec) {
            v[i] = *reinterpret_cast<const bf16x8*>(xp + idx * 8);
            g0[i] = *reinterpret_cast<const f32x4*>(gain + idx * 8);
            g1[i] = *reinterpret_cast<const f32x4*>(gain + idx * 8 + 4);
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (lane + 64 * i < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sq += (float)v[i][e] * (float)v[i][e];
        }
    }
    const float r = rsqrtf(wave_sum(sq) / (float)C + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + 64 * i;
        if (idx < nvec) {
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[e] = (bf16)((float)v[i][e] * r * g0[i][e]);
                o[e + 4] = (bf16)((float)v[i][e + 4] * r * g1[i][e]);
            }
            *reinterpret_cast<bf16x8*>(xp + idx * 8) = o;
        }
    }
}

// ------------------------------------------------------------------ q/k RMSNorm + RoPE + append, and V^T append
// Blocks [0, norm_blocks): one wave per token.  A lane reads 16 bytes (four rotation pairs) of q and of k per
// step, four heads per wave load, keeps the row in registers (IT steps: C <= 512 IT), reduces the sums of squares over
// the whole row, then normalises, rotates and writes q to its buffer and k to the token's ring slot.  Lane j forms the
// rotation of pair j, angle, sine and cosine in double, so that what is rounded to single precision is exact for any stream
// length (a single-precision sincos, even of the exactly reduced angle, is off by its own last bit); the lanes pick up
// their four by shuffle.  Few tokens: a chain of latencies (load, sum, rotate, store), so only what the row needs is
// compiled in, and the rotation is formed while the row is on its way.
// Blocks [norm_blocks, ...): one (64-token tile, head) each: v goes through LDS and is written
// transposed into the V^T cache, a slot's column given by vt_column.
constexpr int VT_TOK = 64;
constexpr int VT_LD = kHeadDim + 2;     // LDS row stride in elements: odd number of words, no bank conflicts

// Tile of up to 64 tokens (n of them, rows of ld elements at src) of one head into the V^T cache of st; tok0 = index of
// the first token in the append that starts at ring position ring0.  quads: tokens 4 q .. 4 q + 3 sit in four consecutive columns (their slots start at a multiple of four),
// so a lane stores four of them at once, sixteen lanes a row of 128 bytes; else token by token.
__device__ __forceinline__ void append_vt_tile(const bf16* src, size_t ld, int n, const AppendStream& st, int h, int tok0,
                                               int ring0, int S, int W, bool quads, bf16* tile) {
    // all loads of a thread at once (behind a test of the row, or in a loop with the LDS writes, each waits for the one before);
    // rows past the end are copies of the last, which nobody reads.  Text of 512 tokens,
    // 12 heads, 30 layers: 517 -> 488 us together with the keys' gains fetched ahead of their sum.
    constexpr int kLoads = VT_TOK * 16 / 256;
    const int tok_own = threadIdx.x >> 4, c = threadIdx.x & 15;
    bf16x8 own[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) own[i] = *reinterpret_cast<const bf16x8*>(src + (size_t)min(tok_own + 16 * i, n - 1) * ld + c * 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        bf16x2* dst = reinterpret_cast<bf16x2*>(tile + (tok_own + 16 * i) * VT_LD + c * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e] = bf16x2{own[i][2 * e], own[i][2 * e + 1]};
    }
    __syncthreads();
    bf16* const vo = st.vt_cache + (size_t)h * kHeadDim * st.cap;
    if (quads) {
        const int q = threadIdx.x & 15, first = threadIdx.x >> 4;
        if (4 * q >= n) return;
        bf16* const col = vo + vt_column(slot_of(tok0 + 4 * q, ring0, S, W));
        const bool whole = 4 * q + 4 <= n;
#pragma unroll
        for (int i = 0; i < kHeadDim / 16; ++i) {
            const int d = first + 16 * i;
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = tile[(4 * q + e) * VT_LD + d];
            if (whole) *reinterpret_cast<bf16x4*>(col + (size_t)d * st.cap) = v;
            else
                for (int e = 0; 4 * q + e < n; ++e) col[(size_t)d * st.cap + e] = v[e];
        }
        return;
    }
    // lane = token, each wave takes 32 of the 128 channels
    const int tok = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (tok < n) {
        bf16* const col = vo + vt_column(slot_of(tok0 + tok, ring0, S, W));
        for (int d = wave * 32; d < wave * 32 + 32; ++d) col[(size_t)d * st.cap] = tile[tok * VT_LD + d];
    }
}

template <int IT>
__global__ __launch_bounds__(256) void rope_append_kernel(RopeAppendArgs a, int norm_blocks, int tiles_per_stream) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int C = a.C;
    if ((int)blockIdx.x < norm_blocks) {
        // What bounds a chunk here is a chain of latencies, so every load that does not depend on another goes out first: the row
        // without tests of the head (past the end: the last head again), the rotation's tables, and the gains of kAhead steps,
        // which came after the row's sums before; the row is uniform, so that its divisions and its stream's arguments are scalar.
        // 1024 tokens of 12 heads 7.4 -> 6.7 us, of 40 heads 18.9 -> 14.8; fewer and more tokens, and every width, gain as well.
        constexpr int kAhead = IT < 3 ? IT : 3;
        const int row = blockIdx.x * 4 + wave;               // over B * L
        if (row >= a.B * a.L) return;
        const bf16* qp = a.qkv + (size_t)row * 3 * C;
        const bf16* kp = qp + C;
        // a wave load covers four heads: lane l holds pairs 4 (l % 16) .. + 3 of head l / 16 + 4 it
        const int hl = lane >> 4;
        const int p0 = 4 * (lane & 15);                      // first of this lane's four rotation pairs
        const int axis = a.pair_axis[lane];
        const double inv_freq = a.inv_freq[lane];
        bf16x8 qv[IT], kv[IT];
        f32x4 gain[IT][4];
        auto column = [&](int it) { return min(hl + 4 * it, a.H - 1) * kHeadDim + 2 * p0; };
        auto fetch_gain = [&](int it) {
            const int c = column(it);
            gain[it][0] = *reinterpret_cast<const f32x4*>(a.g_q + c);
            gain[it][1] = *reinterpret_cast<const f32x4*>(a.g_q + c + 4);
            gain[it][2] = *reinterpret_cast<const f32x4*>(a.g_k + c);
            gain[it][3] = *reinterpret_cast<const f32x4*>(a.g_k + c + 4);
        };
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            qv[it] = *reinterpret_cast<const bf16x8*>(qp + column(it));
            kv[it] = *reinterpret_cast<const bf16x8*>(kp + column(it));
        }
#pragma unroll
        for (int it = 0; it < kAhead; ++it) fetch_gain(it);
        __builtin_amdgcn_sched_barrier(0);
        const int b = row / a.L;
        const int i = row - b * a.L;
        const AppendStream& st = a.st[b];
        // position of the token; lane j forms the rotation of pair j, then every lane fetches its four
        const int frame = (a.desc ? a.desc->frame_pos0[b] : st.frame_pos0) + i / a.tokens_per_frame;
        const int inside = i % a.tokens_per_frame;
        const int pos = axis == 0 ? frame : (axis == 1 ? inside / a.grid_w : inside % a.grid_w);
        double sn, cs;
        sincos((double)pos * inv_freq, &sn, &cs);
        const float cf_own = (float)cs, sf_own = (float)sn;
        float cf[4], sf[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            cf[e] = __shfl(cf_own, p0 + e, kWave);
            sf[e] = __shfl(sf_own, p0 + e, kWave);
        }
        const long long g = (a.desc ? a.desc->g0[b] : st.g0) + i;
        const int slot = slot_of(i, a.desc ? a.desc->ring0[b] : st.ring0, a.S, a.W);
        float sq = 0.0f, sk = 0.0f;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            if (hl + 4 * it < a.H) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    sq += (float)qv[it][e] * (float)qv[it][e];
                    sk += (float)kv[it][e] * (float)kv[it][e];
                }
            }
        }
        const float rq = rsqrtf(wave_sum(sq) / (float)C + a.eps);
        const float rk = rsqrtf(wave_sum(sk) / (float)C + a.eps);
        if (lane == 0) st.ids[slot] = g;
        bf16* qo = a.q_out + (size_t)row * C;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int h = hl + 4 * it;
            if (it + kAhead < IT) fetch_gain(it + kAhead);
            if (h < a.H) {
                const int c = h * kHeadDim + 2 * p0;
                const f32x4 gq0 = gain[it][0], gq1 = gain[it][1], gk0 = gain[it][2], gk1 = gain[it][3];
                bf16x8 qr, kr;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float gqa = e < 2 ? gq0[2 * e] : gq1[2 * e - 4], gqb = e < 2 ? gq0[2 * e + 1] : gq1[2 * e - 3];
                    const float gka = e < 2 ? gk0[2 * e] : gk1[2 * e - 4], gkb = e < 2 ? gk0[2 * e + 1] : gk1[2 * e - 3];
                    const float q0 = (float)qv[it][2 * e] * rq * gqa, q1 = (float)qv[it][2 * e + 1] * rq * gqb;
                    const float k0 = (float)kv[it][2 * e] * rk * gka, k1 = (float)kv[it][2 * e + 1] * rk * gkb;
                    qr[2 * e] = (bf16)(q0 * cf[e] - q1 * sf[e]);
                    qr[2 * e + 1] = (bf16)(q0 * sf[e] + q1 * cf[e]);
                    kr[2 * e] = (bf16)(k0 * cf[e] - k1 * sf[e]);
                    kr[2 * e + 1] = (bf16)(k0 * sf[e] + k1 * cf[e]);
                }
                *reinterpret_cast<bf16x8*>(qo + c) = qr;
                *reinterpret_cast<bf16x8*>(st.k_cache + ((size_t)h * st.cap + slot) * kHeadDim + 2 * p0) = kr;
            }
        }
        return;
    }
    // ---- V^T tiles
    __shared__ bf16 tile[VT_TOK * VT_LD];
    const int vb = blockIdx.x - norm_blocks;
    const int h = vb % a.H;
    const int tile_id = vb / a.H;
    const int b = tile_id / tiles_per_stream;
    const int tok0 = (tile_id - b * tiles_per_stream) * VT_TOK;
    append_vt_tile(a.qkv + ((size_t)b * a.L + tok0) * 3 * C + 2 * C + h * kHeadDim, (size_t)3 * C, min(VT_TOK, a.L - tok0), a.st[b], h,
                   tok0, a.desc ? a.desc->ring0[b] : a.st[b].ring0, a.S, a.W, a.tokens_per_frame % 4 == 0, tile);
}

// ------------------------------------------------------------------ append of rows without rotation
// NORM: text keys, RMSNorm-ed on the way, their gains fetched with the row instead of after its sum; final keys have none.
// Beyond 40 heads only the first gains are, the others four steps ahead, and the row stays in 16 bits across its sum: with all
// of them, and with registers for gains in the append of final keys too, a workgroup had a unit to itself (282 registers).
// Gains after the sum -> all ahead for either kind -> this: text of 1560 x 48 heads 14.9 -> 21.2 -> 14.1 us, of 512 x 64 heads
// 14.0 -> 8.9 -> 8.6; final keys of 1024 x 64 heads 11.4 -> 12.7 -> 10.6 us, of 1024 x 12 heads 3.9 -> 3.7 -> 3.8.
template <int IT, bool NORM>
__global__ __launch_bounds__(256) void plain_append_kernel(PlainAppendArgs a, int k_blocks) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int C = a.C;
    if ((int)blockIdx.x < k_blocks) {
        const int row = blockIdx.x * 4 + wave;
        if (row >= a.n) return;
        const int hl = lane >> 4, c0 = 8 * (lane & 15);      // a wave load covers four heads
        auto column = [&](int it) { return min(hl + 4 * it, a.H - 1) * kHeadDim + c0; };          // past the end: the last head again
        bf16x8 kv[IT];
#pragma unroll
        for (int it = 0; it < IT; ++it) kv[it] = *reinterpret_cast<const bf16x8*>(a.k + (size_t)row * C + column(it));
        const int slot = slot_of(row, a.st.ring0, a.S, a.W);
        constexpr int kAhead = !NORM ? 0 : IT <= 10 ? IT : 4;
        f32x4 gain[IT][2];
        auto fetch_gain = [&](int it) {
            gain[it][0] = *reinterpret_cast<const f32x4*>(a.g_k + column(it));
            gain[it][1] = *reinterpret_cast<const f32x4*>(a.g_k + column(it) + 4);
        };
        float r = 1.0f;
        if constexpr (NORM) {
#pragma unroll
            for (int it = 0; it < kAhead; ++it) fetch_gain(it);
            __builtin_amdgcn_sched_barrier(0);
            float sq = 0.0f;
#pragma unroll
            for (int it = 0; it < IT; ++it)
                if (hl + 4 * it < a.H)
#pragma unroll
                    for (int e = 0; e < 8; ++e) sq += (float)kv[it][e] * (float)kv[it][e];
            r = rsqrtf(wave_sum(sq) / (float)C + a.eps);
            if (kAhead < IT)
#pragma unroll
                for (int it = 0; it < IT; ++it) asm volatile("" : "+v"(kv[it]));        // the row stays in 16 bits across its sum
        }
        if (lane == 0 && a.st.ids != nullptr) a.st.ids[slot] = a.st.g0 + row;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int h = hl + 4 * it;
            if (NORM && it + kAhead < IT) fetch_gain(it + kAhead);
            if (h < a.H) {
                if constexpr (NORM) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        kv[it][e] = (bf16)((float)kv[it][e] * r * gain[it][0][e]);
                        kv[it][e + 4] = (bf16)((float)kv[it][e + 4] * r * gain[it][1][e]);
                    }
                }
                *reinterpret_cast<bf16x8*>(a.st.k_cache + ((size_t)h * a.st.cap + slot) * kHeadDim + c0) = kv[it];
            }
        }
        // a cache may have more heads than a model's 64 (final keys only: text keys belong to a model)
        for (int h = hl + 4 * IT; h < a.H; h += 4)
            *reinterpret_cast<bf16x8*>(a.st.k_cache + ((size_t)h * a.st.cap + slot) * kHeadDim + c0) =
                *reinterpret_cast<const bf16x8*>(a.k + (size_t)row * C + h * kHeadDim + c0);
        return;
    }
    __shared__ bf16 tile[VT_TOK * VT_LD];
    const int vb = blockIdx.x - k_blocks;
    const int h = vb % a.H;
    const int tok0 = (vb / a.H) * VT_TOK;
    append_vt_tile(a.v + (size_t)tok0 * C + h * kHeadDim, (size_t)C, min(VT_TOK, a.n - tok0), a.st, h, tok0, a.st.ring0, a.S, a.W,
                   a.quads != 0, tile);
}

// ------------------------------------------------------------------ conditioning
struct TimestepArgs {
    float t[kMaxBatch];
};

__global__ void timestep_embedding_kernel(TimestepArgs ts, const StepDesc* desc, float* emb, int B, int t_dim,
                                          double log2_base) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= B * t_dim) return;
    const int b = idx / t_dim;
    const int j = idx - b * t_dim;
    const int half = t_dim / 2;
    const int jj = j < half ? j : j - half;
    const double w = exp2(-log2_base * (double)jj / (double)half);
    const double arg = (double)(desc ? desc->timestep[b] : ts.t[b]) * w;
    emb[idx] = (float)(j < half ? cos(arg) : sin(arg));
}

// y[b][n] = sum_k act(x[b][k]) W[n][k] + bias[n] for up to NB rows x.  Bound by the weight stream (the modulation
// projection of the 14B model is 315 MB).  The activated inputs go through LDS, GEMV_K of them at a time, formed once per
// workgroup; a wave owns R weight rows at a time, so that an input read from LDS serves R of them.  (One wave per row that
// formed the activation itself, eight exponentials per eight weights, ran at 1.07 TB/s: 293 us.)  The R NB sums are
// reduced by halving: at every step a lane keeps half of the values and sends the other half.
constexpr int GEMV_K = 1024;
template <int NB, int R>
__global__ __launch_bounds__(256) void gemv_kernel(const float* x, const bf16* w, const float* bias, float* y, int B, int N,
                                                   int K, int silu_in) {
    __shared__ __attribute__((aligned(16))) float xs[NB][GEMV_K];
    const int lane = threadIdx.x & 63;
    const int n0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
    float acc[R * NB];
#pragma unroll
    for (int i = 0; i < R * NB; ++i) acc[i] = 0.0f;
    for (int k0 = 0; k0 < K; k0 += GEMV_K) {
        const int kn = min(GEMV_K, K - k0);                   // a multiple of 8
        bf16x8 wv[GEMV_K / 512][R];
#pragma unroll
        for (int c = 0; c < GEMV_K / 512; ++c) {
            const int k = min(512 * c + lane * 8, kn - 8);
#pragma unroll
            for (int r = 0; r < R; ++r) wv[c][r] = *reinterpret_cast<const bf16x8*>(w + (size_t)min(n0 + r, N - 1) * K + k0 + k);
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            for (int k = threadIdx.x; k < kn; k += 256) {
                float v = b < B ? x[(size_t)b * K + k0 + k] : 0.0f;
                if (silu_in) v = silu_f(v);
                xs[b][k] = v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < GEMV_K / 512; ++c) {
            const int k = 512 * c + lane * 8;
            if (k < kn) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const f32x4 x0 = *reinterpret_cast<const f32x4*>(&xs[b][k]), x1 = *reinterpret_cast<const f32x4*>(&xs[b][k + 4]);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[r * NB + b] += x0[e] * (float)wv[c][r][e];
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[r * NB + b] += x1[e] * (float)wv[c][r][e + 4];
                    }
                }
            }
        }
    }
    int index = 0, off = 32;
#pragma unroll
    for (int s = R * NB / 2; s >= 1; s /= 2, off /= 2) {
        const bool upper = (lane & off) != 0;
#pragma unroll
        for (int i = 0; i < s; ++i) {
            const float keep = upper ? acc[i + s] : acc[i], send = upper ? acc[i] : acc[i + s];
            acc[i] = keep + __shfl_xor(send, off, kWave);
        }
        index += upper ? s : 0;
    }
    const int tail = off;                                     // lanes that differ below bit `off` hold parts of one sum
    for (; off >= 1; off /= 2) acc[0] += __shfl_xor(acc[0], off, kWave);
    const int n = n0 + index / NB, b = index % NB;
    if ((tail == 0 || (lane & (2 * tail - 1)) == 0) && n < N && b < B) y[(size_t)b * N + n] = acc[0] + bias[n];
}

}  // namespace

template <bool EARLY>
static hipError_t launch_layernorm_t(const LnArgs& a, hipStream_t s) {
    const dim3 grid((a.rows + 1) / 2), block(256);
    const int nv = (a.C + 511) / 512;                   // float4 values per lane: 128 lanes per row
    if (nv <= 1) hipLaunchKernelGGL((layernorm_kernel<1, EARLY>), grid, block, 0, s, a);
    else if (nv <= 3) hipLaunchKernelGGL((layernorm_kernel<3, EARLY>), grid, block, 0, s, a);
    else if (nv <= 4) hipLaunchKernelGGL((layernorm_kernel<4, EARLY>), grid, block, 0, s, a);
    else if (nv <= 6) hipLaunchKernelGGL((layernorm_kernel<6, EARLY>), grid, block, 0, s, a);
    else if (nv <= 10) hipLaunchKernelGGL((layernorm_kernel<10, EARLY>), grid, block, 0, s, a);
    else if (nv <= 16) hipLaunchKernelGGL((layernorm_kernel<16, EARLY>), grid, block, 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_layernorm(const LnArgs& a, hipStream_t s) {
    return a.rows <= 4096 ? launch_layernorm_t<true>(a, s) : launch_layernorm_t<false>(a, s);
}

hipError_t launch_rmsnorm_inplace(bf16* x, const float* gain, int rows, int C, int ld, float eps, hipStream_t s) {
    const dim3 grid((rows + 3) / 4), block(256);
    const int nv = (C + 511) / 512;                     // 16-byte pieces per lane
    if (nv <= 1) hipLaunchKernelGGL(rmsnorm_inplace_kernel<1>, grid, block, 0, s, x, gain, rows, C, ld, eps);
    else if (nv <= 3) hipLaunchKernelGGL(rmsnorm_inplace_kernel<3>, grid, block, 0, s, x, gain, rows, C, ld, eps);
    else if (nv <= 6) hipLaunchKernelGGL(rmsnorm_inplace_kernel<6>, grid, block, 0, s, x, gain, rows, C, ld, eps);
    else if (nv <= 10) hipLaunchKernelGGL(rmsnorm_inplace_kernel<10>, grid, block, 0, s, x, gain, rows, C, ld, eps);
    else if (nv <= 16) hipLaunchKernelGGL(rmsnorm_inplace_kernel<16>, grid, block, 0, s, x, gain, rows, C, ld, eps);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// F(IT) with the smallest compiled number of 512-channel steps that covers H heads (the largest, 64 heads, beyond)
#define SDV2_BY_STEPS(H, F)                         \
    do {                                            \
        const int steps__ = ((H) + 3) / 4;          \
        if (steps__ <= 1) F(1);                     \
        else if (steps__ <= 2) F(2);                \
        else if (steps__ <= 3) F(3);                \
        else if (steps__ <= 4) F(4);                \
        else if (steps__ <= 6) F(6);                \
        else if (steps__ <= 8) F(8);                \
        else if (steps__ <= 10) F(10);              \
        else F(16);                                 \
    } while (0)

hipError_t launch_rope_append(const RopeAppendArgs& a, hipStream_t s) {
    const int norm_blocks = (a.B * a.L + 3) / 4;
    const int tiles_per_stream = (a.L + VT_TOK - 1) / VT_TOK;
    const int v_blocks = a.B * tiles_per_stream * a.H;
#define F(IT) hipLaunchKernelGGL(rope_append_kernel<IT>, dim3(norm_blocks + v_blocks), dim3(256), 0, s, a, norm_blocks, tiles_per_stream)
    SDV2_BY_STEPS(a.H, F);
#undef F
    return hipGetLastError();
}

hipError_t launch_plain_append(const PlainAppendArgs& a, hipStream_t s) {
    const int k_blocks = (a.n + 3) / 4;
    const int v_blocks = ((a.n + VT_TOK - 1) / VT_TOK) * a.H;
#define F(IT) hipLaunchKernelGGL((a.g_k != nullptr ? plain_append_kernel<IT, true> : plain_append_kernel<IT, false>), dim3(k_blocks + v_blocks), dim3(256), 0, s, a, k_blocks)
    SDV2_BY_STEPS(a.H, F);
#undef F
    return hipGetLastError();
}

hipError_t launch_text_relayout(const bf16* k_rows, const bf16* v_rows, const float* g_k, float eps, bf16* kt, bf16* vtt, int L_t,
                                int C, int H, int cap, hipStream_t s) {
    // the text K/V buffers are a cache with no ring: slot = token index
    PlainAppendArgs a;
    a.k = k_rows;
    a.v = v_rows;
    a.n = L_t;
    a.C = C;
    a.H = H;
    a.S = cap;          // every token is "sink": slot(g) = g
    a.W = 1;
    a.quads = 1;
    a.g_k = g_k;
    a.eps = eps;
    a.st.k_cache = kt;
    a.st.vt_cache = vtt;
    a.st.ids = nullptr;
    a.st.g0 = 0;
    a.st.ring0 = ring_position(0, cap, 1);
    a.st.frame_pos0 = 0;
    a.st.cap = cap;
    return launch_plain_append(a, s);
}

template <int NB>
static hipError_t launch_gemv_t(const float* x, const bf16* w, const float* bias, float* y, int B, int N, int K, int silu_in,
                                hipStream_t s) {
    // eight rows per wave where that still gives every compute unit a workgroup; else one (timestep MLP: latency)
    if (N >= 8192) hipLaunchKernelGGL((gemv_kernel<NB, 8>), dim3((N + 31) / 32), dim3(256), 0, s, x, w, bias, y, B, N, K, silu_in);
    else hipLaunchKernelGGL((gemv_kernel<NB, 1>), dim3((N + 3) / 4), dim3(256), 0, s, x, w, bias, y, B, N, K, silu_in);
    return hipGetLastError();
}

hipError_t launch_gemv(const float* x, const bf16* w, const float* bias, float* y, int B, int N, int K, int silu_in,
                       hipStream_t s) {
    if (B == 1) return launch_gemv_t<1>(x, w, bias, y, B, N, K, silu_in, s);
    if (B == 2) return launch_gemv_t<2>(x, w, bias, y, B, N, K, silu_in, s);
    if (B <= 4) return launch_gemv_t<4>(x, w, bias, y, B, N, K, silu_in, s);
    return launch_gemv_t<8>(x, w, bias, y, B, N, K, silu_in, s);
}

hipError_t launch_timestep_embedding(const float* t_host, const StepDesc* desc, float* emb, int B, int t_dim, double base,
                                     hipStream_t s) {
    TimestepArgs ts;
    for (int b = 0; b < kMaxBatch; ++b) ts.t[b] = (t_host && b < B) ? t_host[b] : 0.0f;
    const int n = B * t_dim;
    hipLaunchKernelGGL(timestep_embedding_kernel, dim3((n + 255) / 256), dim3(256), 0, s, ts, desc, emb, B, t_dim,
                       log2(base));
    return hipGetLastError();
}

namespace {
__global__ void set_step_desc_kernel(StepDesc d, StepDesc* dst) {
    if (threadIdx.x == 0) *dst = d;
}
}  // namespace

hipError_t launch_set_step_desc(const StepDesc& d, StepDesc* dst, hipStream_t s) {
    hipLaunchKernelGGL(set_step_desc_kernel, dim3(1), dim3(64), 0, s, d, dst);
    return hipGetLastError();
}

}  // namespace sdv2
