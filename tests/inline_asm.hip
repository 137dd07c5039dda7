// The decode kernels' inline-assembly helpers behind the least favourable instruction in front of them: a vector
// instruction (readfirstlane) that wrote the base, or the words, that they are given.  Compiled to assembly by test_inline_asm.py.
#include "decode_mfma.h"

using namespace fairkv;

extern "C" __global__ void stores(float *const *bases, float4 x, float m)
{
    float *base = bases[threadIdx.x / 64];
    publish_f32x4(base, threadIdx.x * 16, x);
}
extern "C" __global__ void small_stores(float *const *bases, float x, float y)
{
    float *base = bases[threadIdx.x / 64];
    publish_f32x2(base, threadIdx.x * 8, x, y);
}
extern "C" __global__ void loads(const float *const *bases, float *out)
{
    __shared__ __attribute__((aligned(1024))) char lds[1024];
    const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FAIRKV_LDS_PTR(lds)));
    load16_to_lds(uniform_ptr(bases[threadIdx.x / 64]), threadIdx.x * 16, at);
    wait_vmcnt<0>();
    out[threadIdx.x] = reinterpret_cast<const float *>(lds)[threadIdx.x];
}
extern "C" __global__ void kept_loads(const float *const *bases, float *out)
{
    __shared__ __attribute__((aligned(1024))) char lds[1024];
    const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FAIRKV_LDS_PTR(lds)));
    load16_to_lds_keep(uniform_ptr(bases[threadIdx.x / 64]), threadIdx.x * 16, at);
    wait_vmcnt<0>();
    out[threadIdx.x] = reinterpret_cast<const float *>(lds)[threadIdx.x];
}
template <int N>
__device__ __forceinline__ void tile(const float *const *bases, float *out)
{
    __shared__ __attribute__((aligned(1024))) char lds[N * 1024];
    const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FAIRKV_LDS_PTR(lds)));
    uint32_t off[N];
    for (int i = 0; i < N; ++i) off[i] = threadIdx.x * 16;
    load_tile_to_lds<N>(uniform_ptr(bases[threadIdx.x / 64]), off, at);
    wait_vmcnt<0>();
    out[threadIdx.x] = reinterpret_cast<const float *>(lds)[threadIdx.x];
}
extern "C" __global__ void tile2(const float *const *bases, float *out) { tile<2>(bases, out); }
extern "C" __global__ void tile4(const float *const *bases, float *out) { tile<4>(bases, out); }

extern "C" __global__ void argument_lanes(const uint32_t *words, uint32_t *out)
{
    uint32_t w[sizeof(CallArgs) / 4];
    for (int i = sizeof(CallArgs) / 4 - 1; i >= 0; --i) {      // the word that is used first is written last
        w[i] = __builtin_amdgcn_readfirstlane(words[i * 64 + threadIdx.x % 64]);
        __builtin_amdgcn_sched_barrier(0);
    }
    CallArgs a;
    __builtin_memcpy(&a, w, sizeof a);
    out[threadIdx.x] = ArgLanes(a).lanes;
}
extern "C" __global__ void factor_lanes(const float *words, float *out)
{
    float k[kScaleHeads], v[kScaleHeads];
    for (int i = kScaleHeads - 1; i >= 0; --i) {
        __builtin_amdgcn_sched_barrier(0);
        k[i] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(words[i * 64 + threadIdx.x % 64])));
    }
    for (int i = 0; i < kScaleHeads; ++i) v[i] = words[i];
    out[threadIdx.x] = lane_values(k, v);
}
