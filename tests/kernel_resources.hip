// Instantiations of the decode kernels that stand for the others (the headline shape with and without the code for short
// pairs and for deep cuts, 16 columns, two 8-bit and an fp32 cache, the vector-ALU kernel), compiled by
// test_kernel_resources.py to read the compiler's resource report: seconds instead of the minutes of the whole library.
#include "decode_f32.h"
#include "decode_mfma.h"
#include "decode_valu.h"
template __global__ void fairkv::fairkv_decode_mfma_kernel<128, 8, false, false, false, false>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_mfma_kernel<128, 8, false, false, true, false>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_mfma_kernel<128, 4, true, true, true, false>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_mfma_kernel<128, 8, true, false, true, false>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_mfma_kernel<128, 16, true, false, true, false>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_mfma_kernel<64, 8, false, true, true, false>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_f32_kernel<128, 8, false>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_f32_kernel<128, 8, true>(fairkv::DecodeArgs);
template __global__ void fairkv::fairkv_decode_valu_kernel<128, 8>(fairkv::DecodeArgs);
