// Motion-aware noise scheduler (StreamDiffusionV2, Section 4.1, "Motion-aware noise scheduler"):
//   d_t    = sqrt(||v_t - v_{t-1}||^2 / (C H W))                      per latent frame,
//   dhat_t = clip(max_{i in {t-k..t}} d_i / sigma, 0, 1),
//   s_t    = lambda [s_max - (s_max - s_min) dhat_t] + (1 - lambda) s_{t-1}.
// The frame differences are one pass over the latents (HBM-bound, a few hundred KB per frame); the recurrence is a
// handful of scalar operations per frame, done in the same launch by one wave so that s_t is there without a round trip.
#include "common.h"

namespace sdv2 {
namespace {

// One workgroup of four waves: d_t from the partial sums (added in double, fixed butterfly), a wave per frame, then on one
// wave the ring of the last k + 1 values, the window maximum, the clip and the moving average, for t = 0 .. T-1 in order.
// The partial sums of all frames and the ring are fetched at once: fetched frame by frame, sixteen frames are sixteen trips
// to memory one after the other (31 us a call; 24 with a launch of its own for this part, 22 like this).
__device__ __forceinline__ void motion_recurrence(const MotionArgs& a, int n_blocks, int lane, int wave) {
    __shared__ float ds[kMotionMaxFrames];
    __shared__ float window[kMotionMaxK + 1];
    float* const ring = a.state + kMotionHeaderFloats;
    const int ring_len = a.k + 1;
    float s = a.state[0];
    int count = __float_as_int(a.state[1]);
    for (int i = threadIdx.x; i < ring_len; i += 256) window[i] = i < count ? ring[i] : 0.0f;
    for (int t = wave; t < a.T; t += 4) {
        double sum = 0.0;
        for (int b = lane; b < n_blocks; b += kWave)
            sum += (double)__hip_atomic_load(a.partial + (size_t)t * n_blocks + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
        if (lane == 0) ds[t] = (float)sqrt(sum / (double)a.n);
    }
    __syncthreads();
    if (wave != 0) return;
    for (int t = 0; t < a.T; ++t) {
        const float d = ds[t];
        // the window: what the ring holds besides the entry that d replaces, and d
        const int have = count < ring_len ? count : ring_len, pos = count % ring_len;
        float mx = d;
        for (int i = lane; i < have; i += kWave)
            if (i != pos) mx = fmaxf(mx, window[i]);
        mx = wave_max(mx);
        ++count;
        const float dhat = fminf(fmaxf(mx / a.sigma, 0.0f), 1.0f);
        s = a.lambda * (a.s_max - (a.s_max - a.s_min) * dhat) + (1.0f - a.lambda) * s;
        if (lane == 0) {
            window[pos] = d;
            ring[pos] = d;
            a.d_out[t] = d;
            a.dhat_out[t] = dhat;
            a.s_out[t] = s;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");       // window[pos] before the next frame's reads
    }
    if (lane == 0) {
        a.state[0] = s;
        a.state[1] = __int_as_float(count);
    }
}

// grid = (kMotionBlocks, T): partial sums of (v_t - v_{t-1})^2 in fp32, one float per workgroup; the workgroup that is
// the last to hand in its sum runs the recurrence.  A second launch for it cost as much as the pass itself.  The sums and
// the ticket (state[2], 0 between calls) are device-scope atomics, which go through to memory: a sum has arrived there
// before its workgroup takes a ticket (the wait on its store), so whoever holds the last ticket reads all of them.
__global__ __launch_bounds__(256) void motion_update_kernel(MotionArgs a) {
    const int t = blockIdx.y;
    const float* cur = a.frames + (size_t)t * a.n;
    const float* prev = t == 0 ? a.prev : a.frames + (size_t)(t - 1) * a.n;
    float acc = 0.0f;
    if (prev != nullptr) {
        const long long stride = (long long)gridDim.x * 256;
        const long long tid = (long long)blockIdx.x * 256 + threadIdx.x;
        if (a.vec4) {
            const f32x4* c4 = reinterpret_cast<const f32x4*>(cur);
            const f32x4* p4 = reinterpret_cast<const f32x4*>(prev);
            for (long long i = tid; i < a.n / 4; i += stride) {
                const f32x4 d = c4[i] - p4[i];
                acc += d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + d[3] * d[3];
            }
        } else {
            for (long long i = tid; i < a.n; i += stride) {
                const float d = cur[i] - prev[i];
                acc += d * d;
            }
        }
    }
    __shared__ float red[4];
    __shared__ int last;
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    unsigned* const ticket = reinterpret_cast<unsigned*>(a.state + 2);
    if (threadIdx.x == 0) {
        __hip_atomic_store(a.partial + (size_t)t * gridDim.x + blockIdx.x, (red[0] + red[1]) + (red[2] + red[3]), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt 0: the sum is in memory
        asm volatile("" ::: "memory");
        const unsigned n = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = n == gridDim.x * gridDim.y - 1;
        if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (last) motion_recurrence(a, gridDim.x, threadIdx.x & 63, threadIdx.x >> 6);
}

__global__ void motion_init_kernel(float* state, int n_floats, float s_init) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_floats) state[i] = i == 0 ? s_init : 0.0f;          // count = 0 has the bit pattern of 0.0f
}

}  // namespace

hipError_t launch_motion_init(float* state, int n_floats, float s_init, hipStream_t s) {
    hipLaunchKernelGGL(motion_init_kernel, dim3((n_floats + 255) / 256), dim3(256), 0, s, state, n_floats, s_init);
    return hipGetLastError();
}

hipError_t launch_motion_update(const MotionArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(motion_update_kernel, dim3(kMotionBlocks, a.T), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace sdv2
