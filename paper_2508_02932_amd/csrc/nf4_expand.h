// Expansion of NF4 weights on the device (see nf4.hip), shared by the stand-alone kernel and by the preparation kernel of the
// NF4 calls, which expands the weight in the same launch.
#pragma once
#include "plora_internal.h"

namespace plora {

// the 16 levels of the format (fp32)
static __constant__ float kNf4Level[16] = {
    -1.0f, -0.6961928009986877f, -0.5250730514526367f, -0.39491748809814453f,
    -0.28444138169288635f, -0.18477343022823334f, -0.09105003625154495f, 0.0f,
    0.07958029955625534f, 0.16093020141124725f, 0.24611230194568634f, 0.33791524171829224f,
    0.44070982933044434f, 0.5626170039176941f, 0.7229568362236023f, 1.0f};

__device__ inline uint32_t nf4_pack_bf16x2(float lo, float hi)
{
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    typedef float v2f __attribute__((ext_vector_type(2)));
    const v2f f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2bf));
}

// One thread per group of 8 elements (4 bytes of indices): a wave reads 256 contiguous bytes of indices and
// writes 1 KB (bf16) or 2 KB (fp32) of contiguous output.  8 groups share a block constant.  Workgroup wg of n_wg; level:
// 16 floats of LDS.
template <bool BF16>
__device__ inline void nf4_expand(const uint32_t *__restrict__ codes, const float *__restrict__ absmax, void *__restrict__ out,
                                  int64_t n_groups, int wg, int n_wg, float *level)
{
    if (threadIdx.x < 16) level[threadIdx.x] = kNf4Level[threadIdx.x];
    __syncthreads();
    const int64_t stride = (int64_t)n_wg * 256;
    for (int64_t g = (int64_t)wg * 256 + threadIdx.x; g < n_groups; g += stride) {
        const uint32_t c = codes[g];
        const float s = absmax[g >> 3];
        float v[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t b = (c >> (8 * j)) & 0xffu;            // byte j: elements 2j (high half) and 2j + 1 (low half)
            v[2 * j] = level[b >> 4] * s;
            v[2 * j + 1] = level[b & 15u] * s;
        }
        if (BF16) {
            uint4 o;
            o.x = nf4_pack_bf16x2(v[0], v[1]); o.y = nf4_pack_bf16x2(v[2], v[3]);
            o.z = nf4_pack_bf16x2(v[4], v[5]); o.w = nf4_pack_bf16x2(v[6], v[7]);
            static_cast<uint4 *>(out)[g] = o;
        } else {
            static_cast<float4 *>(out)[2 * g] = make_float4(v[0], v[1], v[2], v[3]);
            static_cast<float4 *>(out)[2 * g + 1] = make_float4(v[4], v[5], v[6], v[7]);
        }
    }
}

}  // namespace plora
