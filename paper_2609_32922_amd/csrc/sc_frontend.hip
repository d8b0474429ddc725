// Front end of the SC GEMM on the device: fp32 -> int8 symmetric quantisation with the
// row scale and row metric in one pass (Sec. 3.1 PTQ inputs, Sec. 4.2 fused
// quantisation), and the per-row length policy (Sec. 4.4: min-max normalised row
// metric, calibrated thresholds, a ladder of stream lengths).
#include <math.h>

#include "sc_internal.h"

namespace scg {

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}

// max over a 256-thread block (every thread gets the result)
__device__ float block_max_256(float v) {
    __shared__ float part[4];
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    const float r = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    __syncthreads();
    return r;
}

// round half to even, clamp to [-127, 127]; s == 0 gives 0
__device__ __forceinline__ int quant1(float x, float s) {
    if (!(s > 0.0f)) return 0;
    const float q = fminf(fmaxf(rintf(x / s), -127.0f), 127.0f);
    return (int)q;
}
// The same from inv = 1 / s, which takes a fifth of the division's instructions (the divisions
// alone were as long as the memory traffic): y = x inv is within 127 x 2^-22 < 4e-5 of x / s, so both
// round alike unless y lies that close to a half; there, and for whatever is not finite, divide.
__device__ __forceinline__ int quant1(float x, float s, float inv) {
    const float y = x * inv, r = rintf(y);
    if (fabsf(y - r) < 0.4999f && fabsf(r) <= 127.0f) return (int)r;
    return quant1(x, s);
}

enum { Q_ROWS, Q_ROW_MAX, Q_WITH_SCALE };   // scale per row; row maxima only; with the scale given

// A row of K <= 256 NV elements per wave, held in registers: one pass over memory, no barrier.
// Memory-bound: 18464 x 1024 (94 MB) 34 -> 17 us against the block per row below, which reads every
// row twice and divides every element.  VEC: 16-byte loads and 4-byte stores (rows aligned), else 4
// and 1, elements dealt to the lanes in turn.
template <int MODE, int NV, bool VEC>
__global__ __launch_bounds__(256) void k_quant_wave(int rows, int K, const float *__restrict__ X, int64_t ldx,
                                                    int64_t strideX, int8_t *__restrict__ Q, int64_t ldq,
                                                    int64_t strideQ, float *scale, float *rowmax, int64_t strideS) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), b = blockIdx.y, lane = threadIdx.x & 63;
    if (i >= rows) return;
    const float *x = X + (size_t)b * strideX + (size_t)i * ldx;
    float v[4 * NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        if (VEC) {
            const int d = (k * 64 + lane) * 4;
            float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (d < K) t = *reinterpret_cast<const float4 *>(x + d);
            v[4 * k] = t.x;
            v[4 * k + 1] = t.y;
            v[4 * k + 2] = t.z;
            v[4 * k + 3] = t.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int d = (4 * k + j) * 64 + lane;
                v[4 * k + j] = d < K ? x[d] : 0.0f;
            }
        }
    }
    const size_t si = (size_t)b * strideS + i;
    float s;
    if (MODE == Q_WITH_SCALE) {
        s = scale[si];
    } else {
        float m = 0.0f;
#pragma unroll
        for (int k = 0; k < 4 * NV; ++k) m = fmaxf(m, fabsf(v[k]));
        m = wave_max(m);
        s = m / 127.0f;
        if (lane == 0) {
            if (MODE == Q_ROWS) scale[si] = s;
            if (rowmax) rowmax[si] = m;
        }
        if (MODE == Q_ROW_MAX) return;
    }
    const float inv = 1.0f / s;
    int8_t *q = Q + (size_t)b * strideQ + (size_t)i * ldq;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        if (VEC) {
            const int d = (k * 64 + lane) * 4;
            uint32_t w = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) w |= ((uint32_t)quant1(v[4 * k + j], s, inv) & 255u) << (8 * j);
            if (d < K) *reinterpret_cast<uint32_t *>(q + d) = w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int d = (4 * k + j) * 64 + lane;
                if (d < K) q[d] = (int8_t)quant1(v[4 * k + j], s, inv);
            }
        }
    }
}

// Longer rows: one 256-thread block per row, the row read again for the second pass
template <int MODE>
__global__ __launch_bounds__(256) void k_quant_block(int K, const float *__restrict__ X, int64_t ldx, int64_t strideX,
                                                     int8_t *__restrict__ Q, int64_t ldq, int64_t strideQ, float *scale,
                                                     float *rowmax, int64_t strideS) {
    const int i = blockIdx.x, b = blockIdx.y;
    const float *x = X + (size_t)b * strideX + (size_t)i * ldx;
    const size_t si = (size_t)b * strideS + i;
    float s;
    if (MODE == Q_WITH_SCALE) {
        s = scale[si];
    } else {
        float m = 0.0f;
        for (int d = threadIdx.x; d < K; d += 256) m = fmaxf(m, fabsf(x[d]));
        m = block_max_256(m);
        s = m / 127.0f;
        if (threadIdx.x == 0) {
            if (MODE == Q_ROWS) scale[si] = s;
            if (rowmax) rowmax[si] = m;
        }
        if (MODE == Q_ROW_MAX) return;
    }
    const float inv = 1.0f / s;
    int8_t *q = Q + (size_t)b * strideQ + (size_t)i * ldq;
    for (int d = threadIdx.x; d < K; d += 256) q[d] = (int8_t)quant1(x[d], s, inv);
}

// per tensor, pass 2: tensor maximum over the row maxima, scale broadcast to every row
__global__ __launch_bounds__(256) void k_tensor_scale(int rows, const float *src, float *scale,
                                                      int64_t strideS) {
    const int b = blockIdx.x;
    float m = 0.0f;
    for (int i = threadIdx.x; i < rows; i += 256) m = fmaxf(m, src[(size_t)b * strideS + i]);
    m = block_max_256(m);
    const float s = m / 127.0f;
    for (int i = threadIdx.x; i < rows; i += 256) scale[(size_t)b * strideS + i] = s;
}

struct QArgs {
    int batch, rows, K;
    const float *X;
    int64_t ldx, strideX;
    int8_t *Q;
    int64_t ldq, strideQ;
    float *scale, *rowmax;
    int64_t strideS;
};
template <int MODE, int NV>
static void launch_quant_wave(const QArgs &a, bool vec, hipStream_t st) {
    const dim3 grid((unsigned)((a.rows + 3) / 4), (unsigned)a.batch);
    if (vec)
        hipLaunchKernelGGL((k_quant_wave<MODE, NV, true>), grid, dim3(256), 0, st, a.rows, a.K, a.X, a.ldx, a.strideX, a.Q,
                           a.ldq, a.strideQ, a.scale, a.rowmax, a.strideS);
    else
        hipLaunchKernelGGL((k_quant_wave<MODE, NV, false>), grid, dim3(256), 0, st, a.rows, a.K, a.X, a.ldx, a.strideX,
                           a.Q, a.ldq, a.strideQ, a.scale, a.rowmax, a.strideS);
}
template <int MODE>
static hipError_t launch_quant(const QArgs &a, hipStream_t st) {
    // (a row whose last quad would be cut, or that does not start on a quad, takes single elements)
    const bool vec = a.K % 4 == 0 && reinterpret_cast<uintptr_t>(a.X) % 16 == 0 && a.ldx % 4 == 0 && a.strideX % 4 == 0 &&
                     reinterpret_cast<uintptr_t>(a.Q) % 4 == 0 && a.ldq % 4 == 0 && a.strideQ % 4 == 0;
    if (a.K <= 256) launch_quant_wave<MODE, 1>(a, vec, st);
    else if (a.K <= 768) launch_quant_wave<MODE, 3>(a, vec, st);
    else if (a.K <= 1280) launch_quant_wave<MODE, 5>(a, vec, st);
    else if (a.K <= 2048) launch_quant_wave<MODE, 8>(a, vec, st);
    else
        hipLaunchKernelGGL((k_quant_block<MODE>), dim3((unsigned)a.rows, (unsigned)a.batch), dim3(256), 0, st, a.K, a.X,
                           a.ldx, a.strideX, a.Q, a.ldq, a.strideQ, a.scale, a.rowmax, a.strideS);
    return hipGetLastError();
}

hipError_t launch_quantize(int batch, int rows, int K, const float *X, int64_t ldx, int64_t strideX,
                           int per_tensor, int8_t *Q, int64_t ldq, int64_t strideQ, float *scale,
                           float *rowmax, int64_t strideS, hipStream_t st) {
    QArgs a{batch, rows, K, X, ldx, strideX, Q, ldq, strideQ, scale, rowmax, strideS};
    if (!per_tensor) return launch_quant<Q_ROWS>(a, st);
    // (the row maxima, in scale where the caller wants none)
    if (rowmax == nullptr) a.rowmax = scale;
    hipError_t e = launch_quant<Q_ROW_MAX>(a, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tensor_scale, dim3((unsigned)batch), dim3(256), 0, st, rows, a.rowmax, scale,
                       strideS);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_quant<Q_WITH_SCALE>(a, st);
}

// ----------------------------------------------------------------------------
// per-row lengths
// ----------------------------------------------------------------------------
// Every block takes the minimum and maximum over the whole operator call (up to MREG metrics a
// thread, all their loads in flight at once), then the lengths of its own rows: latency-bound,
// and one block per call took 17 us for 18464 rows, most of it in the divisions (4 us now).
constexpr int MREG = 20;
__global__ __launch_bounds__(1024) void k_mp_lengths(int M, const float *metric, int64_t strideM, MpParams p,
                                                     int32_t *L_out, int64_t strideL) {
    __shared__ float pmin[16], pmax[16];
    const int b = blockIdx.x, tid = threadIdx.x;
    const float *g = metric + (size_t)b * strideM;
    float lo = INFINITY, hi = -INFINITY;
    for (int i0 = 0; i0 < M; i0 += MREG * 1024) {
        float v[MREG];
#pragma unroll
        for (int k = 0; k < MREG; ++k) v[k] = g[min(i0 + k * 1024 + tid, M - 1)];
#pragma unroll
        for (int k = 0; k < MREG; ++k) {
            lo = fminf(lo, v[k]);
            hi = fmaxf(hi, v[k]);
        }
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if ((tid & 63) == 0) {
        pmin[tid >> 6] = lo;
        pmax[tid >> 6] = hi;
    }
    __syncthreads();
    lo = pmin[0];
    hi = pmax[0];
    for (int w = 1; w < 16; ++w) {
        lo = fminf(lo, pmin[w]);
        hi = fmaxf(hi, pmax[w]);
    }
    const float range = hi - lo;
    for (int i = blockIdx.y * 1024 + tid; i < M; i += gridDim.y * 1024) {
        const float t = range > 0.0f ? (g[i] - lo) / range : 0.0f;
        int k = p.n - 1;
        for (int j = 0; j < p.n - 1; ++j) {
            if (t >= p.tau[j]) {
                k = j;
                break;
            }
        }
        L_out[(size_t)b * strideL + i] = p.ladder[k];
    }
}

hipError_t launch_mp_lengths(int batch, int M, const float *metric, int64_t strideM,
                             const MpParams &p, int32_t *L_out, int64_t strideL, hipStream_t st) {
    // (a block reads every metric, so their number is bounded.  Lengths that are written over the metrics
    // take one block per operator call: another one would read metrics that are lengths already)
    const uintptr_t m0 = reinterpret_cast<uintptr_t>(metric), l0 = reinterpret_cast<uintptr_t>(L_out);
    const uintptr_t span = ((uintptr_t)(batch - 1) * (uintptr_t)(strideM > strideL ? strideM : strideL) + (uintptr_t)M) * 4;
    const bool apart = m0 >= l0 ? m0 - l0 >= span : l0 - m0 >= span;
    const int most = apart ? 32 : 1, blocks = (M + 1023) / 1024 < most ? (M + 1023) / 1024 : most;
    hipLaunchKernelGGL(k_mp_lengths, dim3((unsigned)batch, (unsigned)blocks), dim3(1024), 0, st, M, metric, strideM, p,
                       L_out, strideL);
    return hipGetLastError();
}

}  // namespace scg
