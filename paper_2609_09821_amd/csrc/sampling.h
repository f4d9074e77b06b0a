// sampling.h -- the last layer's sampling from partial sums in LDS, and small
// helpers shared by the policy kernels.
#pragma once

#include "device_math.h"
#include "launch.h"

namespace im {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr float HALF_LOG_2PI = 0.91893853320467274f;

// ReLU of a packed bf16 pair: a bf16 whose sign bit is set is a negative
// 16-bit integer, so a packed integer max with zero clears exactly the
// negative values (and -0).
typedef short im_s16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t p)
{
    const im_s16x2_t v = __builtin_bit_cast(im_s16x2_t, p);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v, (im_s16x2_t){0, 0}));
}

// Writes n_valid*A consecutive floats from LDS to dst (16-byte stores when dst
// is 16-byte aligned).
template <int NTHR>
__device__ __forceinline__ void copy_rows_out(float *dst, const float *so, int64_t cnt, int tid)
{
    if ((((uintptr_t)dst) & 15) == 0) {
        const int64_t c4 = cnt >> 2;
        for (int64_t v = tid; v < c4; v += NTHR)
            *(f32x4_t *)(dst + 4 * v) = *(const f32x4_t *)(so + 4 * v);
        for (int64_t v = 4 * c4 + tid; v < cnt; v += NTHR) dst[v] = so[v];
    } else {
        for (int64_t v = tid; v < cnt; v += NTHR) dst[v] = so[v];
    }
}

// Sampling of NE envs from partial tiles part [KS][NE][MP] (16-byte units
// XOR-swizzled by env % 8): each of NTHR threads takes one (env, block of four
// actions) at a time.  mean = bias + the partials in slice order; the noise
// comes from Philox; action = mean + sigma z; each env's logp adds its blocks'
// sums in block order.  Mean and action rows [NE][A] and the per-block sums
// [NE][33] follow the partials in LDS.  All threads call it; sig, sbias, slp0
// and senv are in LDS.
template <int NTHR, int NE, int MP, int KS>
__device__ __forceinline__ void sample_rows(const GemmArgs &g, float *part, const float *sig,
                                            const float *sbias, const float &slp0,
                                            const uint32_t *senv, int64_t n0, int64_t nv, int tid)
{
    const int A = g.A;
    float *smean = part + KS * NE * MP;
    float *sact = smean + NE * A;
    float *slp = sact + NE * A;
    const int G = (A + 3) / 4;
    for (int it = tid; it < NE * G; it += NTHR) {
        const int e = it & (NE - 1), j = it / NE;
        if (e >= nv) continue;
        float mu[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) mu[q] = 4 * j + q < A ? sbias[4 * j + q] : 0.0f;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const f32x4_t v = *(const f32x4_t *)(part + (k * NE + e) * MP + 4 * (j ^ (e & 7)));
#pragma unroll
            for (int q = 0; q < 4; ++q) mu[q] += v[q];
        }
        float z[4];
        normals4(g.seed, (uint32_t)(n0 + e), senv[e], (uint32_t)j, 0u, z);
        float lp = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int m = 4 * j + q;
            if (m < A) {
                smean[e * A + m] = mu[q];
                sact[e * A + m] = mu[q] + sig[m] * z[q];
                lp += 0.5f * z[q] * z[q];
            }
        }
        slp[e * 33 + j] = lp;
    }
    __syncthreads();
    if (tid < nv && g.logp) {
        float sum = 0.0f;
        for (int j = 0; j < G; ++j) sum += slp[tid * 33 + j];
        g.logp[n0 + tid] = -(sum + slp0);
    }
    copy_rows_out<NTHR>(g.mean + n0 * A, smean, nv * A, tid);
    copy_rows_out<NTHR>(g.action + n0 * A, sact, nv * A, tid);
}

}  // namespace im
