// Adaptive sink refresh and RoPE refresh of the rolling KV cache (StreamDiffusionV2, Section 4.1, "Adaptive sink and
// RoPE refresh"): alpha_i = cos(h_t, s_i) between one frame of the chunk just appended and every sink frame, the copy
// s_i <- h_t, and the move of all cached keys by a whole number of frames in rotary phase.  All three are single
// passes over parts of one (layer, stream) cache: bound by HBM / L2 bandwidth.
#include "common.h"
#include "refresh_ranges.h"

#include <type_traits>

namespace sdv2 {
namespace {

constexpr int kSimBlock = 256;

// Partial sums of <h, s_i>, |h|^2, |s_i|^2 over the value rows.  V^T is [H][128][cap] with a column permutation inside
// every 16 slots, so element (head, d, token j) of a frame that starts at slot s0 sits in column vt_column(s0 + j).
// grid = (blocks over the H * 128 rows, sink frames), a wave per row; each block writes three doubles, summed in a fixed
// order by the second kernel: the result does not depend on scheduling.
__global__ __launch_bounds__(kSimBlock) void sink_similarity_partial_kernel(SinkSimArgs a) {
    const int sink = blockIdx.y;
    const int sink0 = sink * a.P;
    const int rows = a.H * kHeadDim;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // four partial sums of each kind per lane: a lane owns a whole frame of up to three rows (40 heads), and one sum of all of
    // it is four times as far off as these (alpha before its own rounding, 40 heads of 1560 tokens, rms error against 64
    // bits: 4.1e-8 and 1.1e-8)
    float dots[4] = {}, hhs[4] = {}, sss[4] = {};
    auto add = [&](int e, float x, float y) {
        dots[e] += x * y;
        hhs[e] += x * x;
        sss[e] += y * y;
    };
    // Four consecutive slots that start at a multiple of four sit in four consecutive columns (the permutation
    // moves whole groups of four), so frames that start at multiples of four are read 8 bytes at a time, and eight
    // pieces of both frames per lane are in flight (one round of loads for 2048 tokens).
    const bool quads = (a.P % 4 == 0) && (a.src0 % 4 == 0);
    for (int row = blockIdx.x * (kSimBlock / kWave) + wave; row < rows; row += gridDim.x * (kSimBlock / kWave)) {
        const bf16* v = a.vt + (size_t)row * a.cap;
        if (quads) {
            const int n = a.P / 4;
            for (int q0 = lane; q0 < n; q0 += 8 * kWave) {
                bf16x4 x[8], y[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int q = min(q0 + kWave * u, n - 1);
                    x[u] = *reinterpret_cast<const bf16x4*>(v + vt_column(a.src0 + 4 * q));
                    y[u] = *reinterpret_cast<const bf16x4*>(v + vt_column(sink0 + 4 * q));
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (q0 + kWave * u < n) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) add(e, (float)x[u][e], (float)y[u][e]);
                    }
                }
            }
        } else {
            // two bytes at a time, eight or four of both frames in flight (unconditional: under a condition they go out one
            // by one, past the end the last one again)
            auto pieces = [&](auto count, int c0) {
                constexpr int n = decltype(count)::value;
                bf16 x[n], y[n];
#pragma unroll
                for (int u = 0; u < n; ++u) {
                    const int j = min(c0 + kWave * u + lane, a.P - 1);
                    x[u] = v[vt_column(a.src0 + j)];
                    y[u] = v[vt_column(sink0 + j)];
                }
#pragma unroll
                for (int u = 0; u < n; ++u)
                    if (c0 + kWave * u + lane < a.P) add(u & 3, (float)x[u], (float)y[u]);
            };
            int c0 = 0;
            for (; c0 + 8 * kWave <= a.P; c0 += 8 * kWave) pieces(std::integral_constant<int, 8>{}, c0);
            for (; c0 < a.P; c0 += 4 * kWave) pieces(std::integral_constant<int, 4>{}, c0);
        }
    }
    __shared__ float red[3][kSimBlock / kWave];
    const float dot = wave_sum((dots[0] + dots[1]) + (dots[2] + dots[3]));
    const float hh = wave_sum((hhs[0] + hhs[1]) + (hhs[2] + hhs[3]));
    const float ss = wave_sum((sss[0] + sss[1]) + (sss[2] + sss[3]));
    if (lane == 0) {
        red[0][wave] = dot;
        red[1][wave] = hh;
        red[2][wave] = ss;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = 0.0;
        for (int w = 0; w < kSimBlock / kWave; ++w) t += (double)red[threadIdx.x][w];
        a.partial[((size_t)sink * gridDim.x + blockIdx.x) * 3 + threadIdx.x] = t;
    }
}

// alpha_i = dot / sqrt(|h|^2 |s_i|^2), 0 when a norm is 0.  One wave per sink: lane l adds the partial sums of
// workgroups l, l + 64, ... in double, then the lanes are combined by a fixed butterfly.
__global__ __launch_bounds__(kWave) void sink_similarity_final_kernel(SinkSimArgs a, int n_blocks) {
    const int sink = blockIdx.x;
    const int lane = threadIdx.x;
    double acc[3] = {0.0, 0.0, 0.0};
    for (int b = lane; b < n_blocks; b += kWave) {
        const double* p = a.partial + ((size_t)sink * n_blocks + b) * 3;
        acc[0] += p[0];
        acc[1] += p[1];
        acc[2] += p[2];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] += __shfl_xor(acc[c], off, kWave);
    if (lane == 0) a.alpha[sink] = (acc[1] > 0.0 && acc[2] > 0.0) ? (float)(acc[0] / sqrt(acc[1] * acc[2])) : 0.0f;
}

// s_i <- h_t: the P key rows, value columns and token ids of the frame at slot src0 are copied to the sink frame at
// slot dst0.  Blocks [0, v_blocks) copy four value rows of V^T each (P columns, a wave per row, 8 bytes per lane where the
// frames start at multiples of four slots: 2 bytes at a time the copy ran at 1.8 TB/s) and, in the first of them, the
// ids; the rest copy key rows, 16 bytes per lane and four pieces in flight.  The value rows come first: their few long
// blocks would otherwise be the tail.
constexpr int kCopyPieces = 4;

__global__ __launch_bounds__(256) void refresh_sink_kernel(SinkCopyArgs a, int v_blocks) {
    if ((int)blockIdx.x >= v_blocks) {
        // a head's part of the frame is contiguous rows of sixteen 16-byte pieces
        const unsigned per_head = (unsigned)a.key_tokens * 16u, total = (unsigned)a.key_heads * per_head;
        const unsigned i0 = (blockIdx.x - v_blocks) * (256u * kCopyPieces) + threadIdx.x;
        bf16x8 x[kCopyPieces];
        bf16x8* dst[kCopyPieces];
#pragma unroll
        for (int u = 0; u < kCopyPieces; ++u) {
            const unsigned i = min(i0 + 256u * u, total - 1);
            const unsigned h = i / per_head, c = i - h * per_head;
            bf16* const head = a.k + (size_t)h * a.cap * kHeadDim;
            x[u] = reinterpret_cast<const bf16x8*>(head + (size_t)a.src0 * kHeadDim)[c];
            dst[u] = reinterpret_cast<bf16x8*>(head + (size_t)a.dst0 * kHeadDim) + c;
        }
#pragma unroll
        for (int u = 0; u < kCopyPieces; ++u)
            if (i0 + 256u * u < total) *dst[u] = x[u];
        return;
    }
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;      // (head, d) row of V^T
    bf16* v = a.vt + (size_t)row * a.cap;
    if (a.P % 4 == 0 && a.src0 % 4 == 0 && a.dst0 % 4 == 0) {
        const int n = a.P / 4;
        for (int q0 = lane; q0 < n; q0 += 8 * kWave) {
            bf16x4 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = *reinterpret_cast<const bf16x4*>(v + vt_column(a.src0 + 4 * min(q0 + kWave * u, n - 1)));
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q0 + kWave * u < n) *reinterpret_cast<bf16x4*>(v + vt_column(a.dst0 + 4 * (q0 + kWave * u))) = x[u];
        }
    } else {
        for (int c0 = lane; c0 < a.P; c0 += 8 * kWave) {
            bf16 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = v[vt_column(a.src0 + min(c0 + kWave * u, a.P - 1))];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (c0 + kWave * u < a.P) v[vt_column(a.dst0 + c0 + kWave * u)] = x[u];
        }
    }
    if (blockIdx.x == 0)
        for (int j = threadIdx.x; j < a.P; j += 256) a.ids[a.dst0 + j] = a.ids[a.src0 + j];
}

// Every filled slot's key, heads x frame pairs: (x0, x1) <- (x0 c - x1 s, x0 s + x1 c) with (c, s) the cosine and
// sine of -delta * omega_j, formed in double on the host (there are only kMaxFramePairs of them).
// grid = (filled slots x groups of 4 pairs = 16 bytes, heads), two pieces per thread.
__global__ __launch_bounds__(256) void rotate_keys_kernel(RotateKeysArgs a) {
    const unsigned groups = (unsigned)(a.n_pairs + 3) / 4, total = (unsigned)a.n_slots * groups;
    bf16* const head = a.k + (size_t)blockIdx.y * a.cap * kHeadDim;
    bf16x8* p[2];
    bf16x8 x[2];
    unsigned gq[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const unsigned idx = blockIdx.x * 512u + 256u * u + threadIdx.x;
        const unsigned i = min(idx, total - 1), s = i / groups;
        gq[u] = i - s * groups;
        const int si = a.slot0 + (int)s;
        const int slot = si < a.sink_fill ? si : a.S + (si - a.sink_fill);
        p[u] = reinterpret_cast<bf16x8*>(head + (size_t)slot * kHeadDim) + gq[u];
        x[u] = *p[u];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (blockIdx.x * 512u + 256u * u + threadIdx.x >= total) break;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = 4 * gq[u] + e;
            if (j < a.n_pairs) {
                const float c = a.cs[j], s = a.sn[j];
                const float x0 = (float)x[u][2 * e], x1 = (float)x[u][2 * e + 1];
                x[u][2 * e] = (bf16)(x0 * c - x1 * s);
                x[u][2 * e + 1] = (bf16)(x0 * s + x1 * c);
            }
        }
        *p[u] = x[u];
    }
}

}  // namespace

int sink_similarity_blocks(int H) {
    const int blocks = H * kHeadDim / (kSimBlock / kWave);
    return blocks < 512 ? blocks : 512;
}

hipError_t launch_sink_similarity(const SinkSimArgs& a, hipStream_t s) {
    const int nb = sink_similarity_blocks(a.H);
    hipLaunchKernelGGL(sink_similarity_partial_kernel, dim3(nb, a.m), dim3(kSimBlock), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sink_similarity_final_kernel, dim3(a.m), dim3(kWave), 0, s, a, nb);
    return hipGetLastError();
}

hipError_t launch_refresh_sink(const SinkCopyArgs& all, hipStream_t s) {
    SinkCopyArgs a = all;
    unsigned v_blocks = (unsigned)a.H * kHeadDim / 4;                   // all value rows go with the first range of keys
    hipError_t e = hipSuccess;
    for_refresh_ranges(a.H, a.P, 16, a.H, [&](int h0, int heads, int t0, int tokens) {
        if (e != hipSuccess) return;
        a.k = all.k + ((size_t)h0 * a.cap + t0) * kHeadDim;
        a.key_heads = heads;
        a.key_tokens = tokens;
        const unsigned k_blocks = ((unsigned)heads * (unsigned)tokens * 16u + 256u * kCopyPieces - 1) / (256u * kCopyPieces);
        hipLaunchKernelGGL(refresh_sink_kernel, dim3(k_blocks + v_blocks), dim3(256), 0, s, a, (int)v_blocks);
        e = hipGetLastError();
        v_blocks = 0;
    });
    return e;
}

hipError_t launch_rotate_keys(const RotateKeysArgs& all, hipStream_t s) {
    if (all.n_slots == 0) return hipSuccess;
    RotateKeysArgs a = all;
    const int groups = (a.n_pairs + 3) / 4;
    hipError_t e = hipSuccess;
    for_refresh_ranges(a.H, all.n_slots, groups, kMaxGridRows, [&](int h0, int heads, int slot0, int slots) {
        if (e != hipSuccess) return;
        a.k = all.k + (size_t)h0 * a.cap * kHeadDim;
        a.slot0 = slot0;
        a.n_slots = slots;
        hipLaunchKernelGGL(rotate_keys_kernel, dim3(((unsigned)slots * (unsigned)groups + 511) / 512, heads), dim3(256), 0, s, a);
        e = hipGetLastError();
    });
    return e;
}

}  // namespace sdv2
