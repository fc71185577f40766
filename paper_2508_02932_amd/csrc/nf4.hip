// Dequantisation of a base weight stored as 4-bit NormalFloat (NF4, the storage QLoRA publishes; the
// paper runs packed LoRA on such a base and notes that the LoRA computation is unchanged).
//
// Storage: the weight, flat in memory order, in blocks of 64 elements; per block one fp32 constant
// (the block's largest magnitude), per element a 4-bit index into 16 levels in [-1, 1]; two indices
// per byte, the even element in the high half.  value = level[index] * constant, one fp32
// multiplication, rounded to bf16 (nearest even) when the layer runs in bf16.
//
// On this chip the layer's GEMMs are bound by the matrix cores at fine-tuning batch sizes (tens of
// thousands of tokens), not by the bytes of W, so the weight is expanded once per call into the
// caller's workspace by this streaming kernel (4.5 bits read, 16 written per weight: about 1 % of the
// GEMM's time at 32768 tokens) and the fused GEMM runs on it unchanged, instead of spending vector-ALU
// work inside the GEMM's fetch phases, which are its critical path.
#include "nf4_expand.h"

namespace plora {

template <bool BF16>
__global__ void __launch_bounds__(256) k_nf4_dequant(const uint32_t *__restrict__ codes, const float *__restrict__ absmax,
                                                     void *__restrict__ out, int64_t n_groups)
{
    __shared__ float level[16];
    nf4_expand<BF16>(codes, absmax, out, n_groups, blockIdx.x, gridDim.x, level);
}

int nf4_workgroups(int64_t n_elems)
{
    hipError_t cu_err = hipSuccess;
    const int64_t n_cu = device_cu_count(&cu_err);
    const int64_t blocks = (n_elems / 8 + 255) / 256;
    return (int)(blocks < n_cu * 16 ? blocks : n_cu * 16);       // a few workgroups per compute unit, each looping
}

hipError_t launch_nf4_dequant(const void *codes, const float *absmax, int64_t n_elems, bool bf16, void *out, hipStream_t st)
{
    if (n_elems == 0) return hipSuccess;
    const int64_t n_groups = n_elems / 8;
    const int blocks = nf4_workgroups(n_elems);
    if (blocks < 1) return hipErrorInvalidDevice;
    if (bf16) hipLaunchKernelGGL(k_nf4_dequant<true>, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const uint32_t *>(codes),
                                 absmax, out, n_groups);
    else hipLaunchKernelGGL(k_nf4_dequant<false>, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const uint32_t *>(codes),
                            absmax, out, n_groups);
    return hipGetLastError();
}

}  // namespace plora
