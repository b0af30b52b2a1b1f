// Internal declarations shared by the HIP sources of libsdv2 (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sdv2 {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kHeadDim = 128;
constexpr int kMaxBatch = 8;
constexpr int kLatentChannels = 16;      // VAE latent channels; a token covers 2 x 2 latent positions (64 numbers)

// Column of a V^T cache row that holds slot s: inside every group of 16 slots the two middle groups of four
// trade places (0-3, 8-11, 4-7, 12-15), the order in which the S^T accumulator of the attention kernel holds
// its keys.  The map is its own inverse.
__host__ __device__ __forceinline__ int vt_column(int s) { return (s & ~12) | ((s & 4) << 1) | ((s & 8) >> 1); }

// Sum over the wavefront, in every lane, the lanes 32, 16, 8, 4, 2 and 1 apart added in this order: the half and row swaps,
// then two rotations of a row of 16 lanes (by then its halves, then its quarters, are equal, so a rotation is the exchange)
// and two quad permutations.  All on the vector unit: a shuffle through the LDS crossbar costs about ten times the latency,
// and the row kernels of a single chunk are chains of these.  A sum of shuffles in the same order has the same bits.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float wave_sum(float v) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    v += dpp_f<0x128>(v);        // row_ror:8
    v += dpp_f<0x124>(v);        // row_ror:4
    v += dpp_f<0x4E>(v);         // quad_perm [2, 3, 0, 1]
    return v + dpp_f<0xB1>(v);   // quad_perm [1, 0, 3, 2]
}

// Maximum over the wavefront, in every lane, by the same exchanges (fmaxf: a NaN gives way to a number).
__device__ __forceinline__ float wave_max(float v) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    v = fmaxf(v, dpp_f<0x128>(v));
    v = fmaxf(v, dpp_f<0x124>(v));
    v = fmaxf(v, dpp_f<0x4E>(v));
    return fmaxf(v, dpp_f<0xB1>(v));
}

__device__ __forceinline__ float gelu_tanh_f(float x) {
    // 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)),  u = sqrt(2/pi) (x + 0.044715 x^3).  The exponent is formed
    // directly in base 2 and the quotient is x times the hardware reciprocal (1 ulp): the caller rounds the
    // result to bf16.
    constexpr float k1 = -2.0f * 1.4426950408889634f * 0.7978845608028654f;
    constexpr float k3 = k1 * 0.044715f;
    const float e = __builtin_amdgcn_exp2f(x * fmaf(x * x, k3, k1));
    return x * __builtin_amdgcn_rcpf(1.0f + e);
}

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + __expf(-x)); }

// Memory that a launch soon reads, fetched into the memory-side cache (256 MB, in front of HBM, shared by the chip) by
// workgroups behind an earlier launch's own, on compute units that those leave idle.
constexpr int kUnits = 256;           // compute units
constexpr int kMaxWarmRanges = 4;
struct WarmRange {
    const unsigned char* p;           // a multiple of 16; rows of `pitch` bytes (a multiple of 16), of which the first
    unsigned rows, pitch, columns;    // `columns` columns of 1 KB are fetched
};
struct WarmArgs {
    WarmRange range[kMaxWarmRanges];
    unsigned ranges;                  // 0: nothing to fetch
    unsigned blocks;                  // workgroups that share them
};

// What a launch's last round of workgroups leaves idle: waves of workgroups behind its own, and about how many microseconds.
struct IdleUnits {
    unsigned blocks, waves;           // workgroups, and waves of each
    float us;
};

// Reads the ranges and drops what it has read: a wave takes 1 KB of a row at a time, columns before rows, so the first part of
// every row arrives first.  Sixteen loads of a lane are in flight (128 KB of a unit; with eight, 1 % of a step slower).
__device__ __forceinline__ void warm_memory(const WarmArgs& w, unsigned block) {
    constexpr unsigned kInFlight = 16;
    const unsigned lane = threadIdx.x & 63u, waves = blockDim.x >> 6;
    const unsigned step = w.blocks * waves, wave = __builtin_amdgcn_readfirstlane(block * waves + (threadIdx.x >> 6));
    for (unsigned n = 0; n < w.ranges; ++n) {
        const unsigned char* const p = w.range[n].p;
        const unsigned rows = w.range[n].rows, pitch = w.range[n].pitch, columns = w.range[n].columns;
        const unsigned dc = step / rows, dr = step - dc * rows;
        unsigned c = wave / rows, r = wave - c * rows;
        while (c < columns) {
            uint4 v[kInFlight];
#pragma unroll
            for (unsigned u = 0; u < kInFlight; ++u) {
                const bool in = c < columns;                          // past the end: the first column of the first row
                const size_t at = (size_t)(in ? r : 0u) * pitch + min((in ? c : 0u) * 1024u + lane * 16u, pitch - 16u);
                v[u] = *reinterpret_cast<const uint4*>(p + at);
                c += dc;
                r += dr;
                if (r >= rows) {
                    r -= rows;
                    ++c;
                }
            }
#pragma unroll
            for (unsigned u = 0; u < kInFlight; ++u) asm volatile("" ::"v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
        }
    }
}

// ---------------------------------------------------------------- launchers (host side)
// While launches are profiled (sdv2_prof_begin), the launchers of the matrix kernels leave here which one they took, spelled as a
// profiler prints it.
struct LaunchNote {
    bool on;
    char kernel[96];
};
inline LaunchNote g_launch_note{};
enum GemmEpilogue { kEpiBias = 0, kEpiBiasGelu = 1, kEpiGatedResidual = 2, kEpiResidual = 3,
                    kEpiPartial = 4 /* internal: fp32 partial sums of one k part, no bias */,
                    kEpiGainSquares = 5 /* internal: bf16 gain (A W^T + bias), and sums of (A W^T + bias)^2 over pieces of rows */ };

struct GemmArgs {
    const bf16* a;        // [M, K]
    const bf16* w;        // [N, K]
    const float* bias;    // [N] or null
    void* out;            // bf16 [M, N] (epilogue 0, 1) or fp32 [M, N] (2, 3)
    int M, N, K;
    int epilogue;
    const float* gate_a;  // [N]
    const float* gate_b;  // [(M / rows_per_gate), gate_b_stride]
    int gate_b_stride;
    int rows_per_gate;
    // Optional scratch for shapes whose plan splits the k range over several workgroups per tile (null: never
    // split): room for splitk_floats fp32 partial sums.  A second, elementwise kernel adds the parts in k order
    // and applies the epilogue, so the result does not depend on scheduling.
    float* splitk_partials;
    size_t splitk_floats;
    // Optional second product of the same A, shape and epilogue (0 or 1), computed in the same launch: half the tiles are
    // too few for the chip where one is.  Null: none.
    const bf16* w2;
    const float* bias2;
    void* out2;
    // kEpiGainSquares: gain [N] and the sums, [pieces][M].
    const float* gain;
    float* squares;
    bool cold_weights;    // the weights are not in the memory-side cache: each layer has its own, and they exceed it
};
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s);
// The projection in front of an RMSNorm over its N columns with this gain, whose consumer multiplies by the row's factor
// itself: out = gain (A W^T + bias), and the rows' sums of squares in gemm_square_pieces pieces (at most N / 16), [pieces][M]
// at g.squares.  No pieces: the plan of this shape cannot (a k split, the register-staged kernel).
int gemm_square_pieces(const GemmArgs& g);
hipError_t launch_gemm_gain_squares(const GemmArgs& g, hipStream_t s);
// fp32 partial sums the planned launch of an [M, K] x [N, K] product needs (0: its plan does not split k)
size_t gemm_splitk_floats(int M, int N, int K, int epilogue);
// the most that the planned launch of any product of at most M rows, N columns and K needs; grows with each
size_t gemm_splitk_floats_bound(int M, int N, int K);
// Name of the kernel instantiation the plan picks for a shape, spelled as a profiler prints it (benchmark only).
void gemm_plan_name(int M, int N, int K, int epilogue, char* out, size_t cap);
// The plan of a call with `bytes` of scratch: configuration (0: register-staged kernel), k parts, estimated microseconds.
void gemm_plan(int M, int N, int K, int epilogue, int products, size_t bytes, int* tile, int* parts, float* us);
// Tuning hooks (tests and sweeps): a tile plan that replaces the planner's for every shape; false if not understood.
bool set_gemm_tile_override(const char* spec);

// What changes from one denoising step to the next, kept in device memory when the step is replayed from a captured
// graph (the kernels then read it from there instead of from their by-value arguments).
struct StepDesc {
    long long g0[kMaxBatch];          // token id of the chunk's first token, per stream of the call
    int ring0[kMaxBatch];             // its ring position (ring_position)
    int frame_pos0[kMaxBatch];        // RoPE frame index of the chunk's first frame
    int kv_len[kMaxBatch];            // resident slots after the append
    float timestep[kMaxBatch];
};

// Division of n by d as the high half of one product, exact while n d < 2^32 (m = 0 beyond that, and for d = 1).  A division
// in software is a chain of some forty instructions, and a kernel's first addresses wait for several of them.
struct FastDiv {
    unsigned d, m;
};
inline FastDiv fast_div(unsigned d, unsigned long long n_max) {
    return FastDiv{d, d > 1 && n_max * d < (1ull << 32) ? (unsigned)((1ull << 32) / d) + 1u : 0u};
}
__device__ __forceinline__ unsigned divide(unsigned n, const FastDiv& f) {
    if (f.m != 0) return __umulhi(n, f.m);
    return f.d == 1 ? n : n / f.d;
}

struct AttnArgs {
    const bf16* q;                    // [B, L, C]
    const bf16* k[kMaxBatch];         // [H][cap][128]
    const bf16* vt[kMaxBatch];        // [H][128][cap]
    int kv_len[kMaxBatch];
    int cap[kMaxBatch];
    bf16* o;                          // [B, L, C]
    int B, L, H;
    float* part_o;                    // workspace: [splits][B*L][C] fp32
    float* part_ml;                   // workspace: [splits][B*L][H][2] fp32
    int splits;                       // set by plan_attention
    const StepDesc* desc;             // null: kv_len above; else kv_len is read from the device descriptor
    FastDiv by_q_tiles, by_heads;     // set by the launcher, as is the number of workgroups
    unsigned n_wg;
    // Queries whose RMSNorm over C is still to be divided out: the factor of a query's row is one number, so it joins the scale
    // of its scores.  Sums of squares [q_pieces][B L] of the row before its gain (null: the queries are final).
    const float* q_squares;
    int q_pieces;
    float q_eps;
};
// What the host keeps of a launch beside the kernel's arguments.
struct AttnLaunch : AttnArgs {
    int full_kv;                      // the keys of a full cache, of which kv_len are there (0: there will be no more)
    int waves;                        // set by plan_attention: 4 or 8 per workgroup; 2: the key-split form (splits = 1)
    float us;                         // its estimate of the launch
};
void plan_attention(AttnLaunch* a);   // from B, L, H, kv_len, cap and full_kv; what follows here takes a planned launch
IdleUnits attention_idle_units(const AttnLaunch& a);
// Tuning hooks: waves per workgroup (4, 8; 0 = planner) and key-range splits (0 = planner); -1 leaves a value as is.
void set_attention_overrides(int waves, int splits);
size_t attention_workspace_bytes(int B, int L, int C, int max_kv_len);
// the most that a call of at most B streams of at most L queries needs; grows with B, L and max_kv_len
size_t attention_workspace_bytes_bound(int B, int L, int C, int max_kv_len);
// part 1: the kernel; 2: the merge pass only.  warm: what units that the kernel leaves idle fetch meanwhile (null: nothing).
hipError_t launch_attention(const AttnLaunch& a, hipStream_t s, int part = 0, const WarmArgs* warm = nullptr);
inline bool attention_has_merge_pass(const AttnLaunch& a) { return a.splits > 1; }
void attention_plan_name(const AttnLaunch& a, char* out, size_t cap);

// LayerNorm over C with an affine that is either adaLN modulation or a plain (gamma, beta).
struct LnArgs {
    const float* x;       // [rows, C]
    bf16* out;            // [rows, C]
    int rows, C;
    float eps;
    // scale = 1 + (scale_a[c] + scale_b[stream * b_stride + c]) when modulated, gamma[c] otherwise
    const float* scale_a;
    const float* scale_b; // null: plain affine (scale_a = gamma, shift_a = beta)
    const float* shift_a;
    const float* shift_b;
    int b_stride;
    int rows_per_stream;
};
hipError_t launch_layernorm(const LnArgs& a, hipStream_t s);

// launch_gemm for a residual epilogue (2 or 3) whose output x is the input of a LayerNorm that follows it: when the
// plan splits k, the pass that adds the parts owns whole rows and also writes that LayerNorm's output (ln.x is
// ignored: the rows are g.out's; ln.rows = g.M, ln.C = g.N).  *ln_done tells whether it did; if not, the caller
// launches the LayerNorm itself.
// part 0: everything; 1: only the kernel on the matrix cores; 2: only the pass that adds the k parts.
hipError_t launch_gemm_then_layernorm(const GemmArgs& g, const LnArgs& ln, bool* ln_done, hipStream_t s, int part = 0);
// warm: what part 1 fetches on the side (null: nothing).
hipError_t launch_gemm_part(const GemmArgs& g, hipStream_t s, int part, const WarmArgs* warm = nullptr);
IdleUnits gemm_idle_units(const GemmArgs& g);        // of the matrix part
bool gemm_fetches_own_weights(const GemmArgs& g);    // in large pieces, before its k loop gets to them
bool gemm_splits_k(const GemmArgs& g);               // whether the planned launch has such a second pass

// In-place RMSNorm over C of bf16 rows, times gain.
hipError_t launch_rmsnorm_inplace(bf16* x, const float* gain, int rows, int C, int ld, float eps, hipStream_t s);

// q/k RMSNorm + 3D-RoPE + append of k and v into the rolling cache.
struct AppendStream {
    bf16* k_cache;        // [H][cap][128]
    bf16* vt_cache;       // [H][128][cap]
    long long* ids;       // [cap]
    long long g0;         // token id of the chunk's first token
    int ring0;            // its ring position (ring_position)
    int frame_pos0;
    int cap;
};
// Position in the ring of W slots behind a sink of S slots of the token with id g0; negative while it still belongs to
// the sink.  Formed once per append (a 64-bit remainder), so that a kernel finds token g0 + i (i < W) by slot_of.
__host__ __device__ __forceinline__ int ring_position(long long g0, int S, int W) {
    return g0 < S ? (int)(g0 - S) : (int)((g0 - S) % W);
}
__device__ __forceinline__ int slot_of(int i, int ring0, int S, int W) {
    const int r = ring0 + i;
    return S + (r >= W ? r - W : r);
}
struct RopeAppendArgs {
    const bf16* qkv;      // [B*L, 3C]   (or separate k, v when q_out == null)
    bf16* q_out;          // [B*L, C]
    const float* g_q;
    const float* g_k;
    int B, L, C, H;
    int tokens_per_frame, grid_w;
    int S, W;
    float eps;
    double inv_freq[kHeadDim / 2];    // rotation frequency of each pair of a head
    int pair_axis[kHeadDim / 2];      // 0 frame, 1 row, 2 col
    AppendStream st[kMaxBatch];
    const StepDesc* desc;             // null: g0 and frame_pos0 of st[]; else they are read from the device descriptor
};
hipError_t launch_rope_append(const RopeAppendArgs& a, hipStream_t s);

// Append of k, v rows [n, C]: final rows (standalone cache call), or keys that still need their RMSNorm (text keys).
struct PlainAppendArgs {
    const bf16* k;        // [n, C]
    const bf16* v;        // [n, C]
    int n, C, H, S, W;
    int quads;            // every fourth token starts at a slot that is a multiple of four
    const float* g_k;     // null: keys are final; else gain of the RMSNorm over C
    float eps;
    AppendStream st;
};
hipError_t launch_plain_append(const PlainAppendArgs& a, hipStream_t s);

// Sink refresh and RoPE refresh of one (layer, stream) cache (Section 4.1).
struct SinkSimArgs {
    const bf16* vt;       // [H][128][cap]
    int H, cap, P;        // P = tokens per frame
    int src0;             // first slot of the frame h_t
    int m;                // sink frames; sink frame i starts at slot i * P
    double* partial;      // [m][blocks][3]
    float* alpha;         // [m]
};
int sink_similarity_blocks(int H);
hipError_t launch_sink_similarity(const SinkSimArgs& a, hipStream_t s);
struct SinkCopyArgs {
    bf16* k;              // [H][cap][128]
    bf16* vt;             // [H][128][cap]
    long long* ids;       // [cap]
    int H, cap, P;
    int src0, dst0;       // first slots of the source frame and of the sink frame
    int key_heads, key_tokens;      // set by the launcher: heads and tokens per head of one launch's keys, from k on
};
hipError_t launch_refresh_sink(const SinkCopyArgs& a, hipStream_t s);
constexpr int kMaxFramePairs = kHeadDim / 2;
struct RotateKeysArgs {
    bf16* k;              // [H][cap][128]
    int H, cap, S;
    int sink_fill;        // filled sink slots [0, sink_fill)
    int n_slots;          // sink_fill + filled window slots [S, S + n_slots - sink_fill)
    int slot0;            // set by the launcher: how many of them come before this launch's n_slots
    int n_pairs;          // leading pairs of a head that belong to the frame axis
    float cs[kMaxFramePairs], sn[kMaxFramePairs];
};
hipError_t launch_rotate_keys(const RotateKeysArgs& a, hipStream_t s);

// Motion-aware noise scheduler (Section 4.1).  Device state: kMotionHeaderFloats header floats (s, frame count as
// int bits, the ticket of the running launch), then the ring of the last k + 1 intensities, then kMotionMaxFrames * kMotionBlocks partial sums.
constexpr int kMotionHeaderFloats = 16;
constexpr int kMotionBlocks = 64;
constexpr int kMotionMaxFrames = 16;
constexpr int kMotionMaxK = 1023;
struct MotionArgs {
    const float* frames;   // [T][n]
    const float* prev;     // [n] or null: the frame before frames[0]
    long long n;
    int T, k, vec4;
    float sigma, lambda, s_min, s_max;
    float* state;
    float* partial;        // [T][kMotionBlocks]
    float* d_out;          // [T]
    float* dhat_out;       // [T]
    float* s_out;          // [T]
};
hipError_t launch_motion_init(float* state, int n_floats, float s_init, hipStream_t s);
hipError_t launch_motion_update(const MotionArgs& a, hipStream_t s);

// RMSNorm of the text key rows [L_t, C] and re-layout of both into the cache layouts.
hipError_t launch_text_relayout(const bf16* k_rows, const bf16* v_rows, const float* g_k, float eps, bf16* kt, bf16* vtt,
                                int L_t, int C, int H, int cap, hipStream_t s);

// y[b][n] = act_out(sum_k act_in(x[b][k]) W[n][k] + bias[n]); x, y fp32; W bf16 [N, K]; B <= kMaxBatch.
hipError_t launch_gemv(const float* x, const bf16* w, const float* bias, float* y, int B, int N, int K,
                       int silu_in, hipStream_t s);
// t_host: the B timesteps (by value into the launch), or null with desc: they are read from the device descriptor
hipError_t launch_timestep_embedding(const float* t_host, const StepDesc* desc, float* emb, int B, int t_dim, double base,
                                     hipStream_t s);
hipError_t launch_set_step_desc(const StepDesc& d, StepDesc* dst, hipStream_t s);
// While set (per thread), the dense launchers only make sure their kernels' attributes are set and launch nothing:
// used once before a stream capture so that no attribute call falls inside it.
void set_attributes_only(bool on);
bool attributes_only();

// Latents <-> tokens, noise rate, sampler update (latent_io.hip).  z, v: fp32 [B][16][F][2 gh][2 gw]; patches bf16 and
// tok fp32 [B F gh gw][64]; n = elements per stream; rate / sigma / sigma_next: host arrays [B].
hipError_t launch_patchify(const float* z, bf16* patches, int B, int F, int gh, int gw, hipStream_t s);
hipError_t launch_unpatchify(const float* tok, float* v, int B, int F, int gh, int gw, hipStream_t s);
hipError_t launch_noise(const float* x, const float* eps, float* out, int B, long long n, const float* rate, hipStream_t s);
hipError_t launch_sampler(const float* z, const float* v, const float* eps, float* z_next, float* x0, int B, long long n,
                          const float* sigma, const float* sigma_next, hipStream_t s);

// Benchmark-only microkernels: a register-resident loop of bf16 matrix instructions (iters x 8 per wave, eight waves
// per workgroup) and a streaming copy of `bytes` (multiple of 16) bytes.
hipError_t launch_peak_mfma(int iters, int workgroups, float* sink, hipStream_t s);
double peak_mfma_flops(int iters, int workgroups);
hipError_t launch_peak_copy(const void* src, void* dst, size_t bytes, hipStream_t s);
hipError_t launch_peak_lds(int iters, const unsigned char* src, float* sink, unsigned long long* ticks, hipStream_t s);

}  // namespace sdv2
