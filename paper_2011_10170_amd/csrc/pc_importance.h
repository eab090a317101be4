// Tap importances of 64 consecutive kernels by one wavefront, shared by selection and pool generation.
#ifndef PC_IMPORTANCE_H
#define PC_IMPORTANCE_H
#include "pc_internal.h"

// The 9 weights and gradients of kernels k0 .. k0 + n - 1 (1 <= n <= 64) on their way from memory, as they lie there: the
// importance of an element needs its own weight and gradient only, so it is formed before the elements go to LDS to be
// regrouped by kernel (one LDS pass for both tensors). A wavefront stages for itself: no barriers, and the wavefronts of a CU
// drift apart, so that some compute while others wait for memory. (With workgroups that staged, waited and ranked together
// all of them asked for memory at once and then computed at once: 2.6 TB/s.)
struct PcImpRegs { float4 w[3], g[3]; };
struct __attribute__((packed, aligned(4))) PcQuad { float x, y, z, w; };   // 4 floats on a 4-byte boundary: one 16-byte access

// The last quad is moved back to end with the last element, and quads past it repeat it: every load is unconditional. Without
// gradients the weights are loaded in their place (pc_imp_put ignores them).
__device__ __forceinline__ void pc_imp_issue(const float *__restrict__ W, const float *__restrict__ G, int64_t k0, int n, PcImpRegs &r)
{
    const int lane = threadIdx.x & 63;
    const float *wsrc = W + k0 * 9, *gsrc = (G ? G : W) + k0 * 9;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int e = (j * 64 + lane) * 4 < n * 9 - 4 ? (j * 64 + lane) * 4 : n * 9 - 4;
        const PcQuad a = *reinterpret_cast<const PcQuad *>(wsrc + e), b = *reinterpret_cast<const PcQuad *>(gsrc + e);
        r.w[j] = make_float4(a.x, a.y, a.z, a.w);
        r.g[j] = make_float4(b.x, b.y, b.z, b.w);
    }
}

// Importances to LDS: element t of kernel k0 + l at s[9 * l + t]. s: 64 * 9 floats of this wavefront, 16-byte aligned.
__device__ __forceinline__ void pc_imp_put(const PcImpRegs &r, bool grad, int n, float *s)
{
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_wave_barrier();            // the reads of the chunk before stay before these writes
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const float x = grad ? r.g[j].x * r.w[j].x : r.w[j].x, y = grad ? r.g[j].y * r.w[j].y : r.w[j].y;
        const float z = grad ? r.g[j].z * r.w[j].z : r.w[j].z, w = grad ? r.g[j].w * r.w[j].w : r.w[j].w;
        const int e = (j * 64 + lane) * 4 < n * 9 - 4 ? (j * 64 + lane) * 4 : n * 9 - 4;
        if ((j * 64 + lane) * 4 < n * 9) {
            const PcQuad q = {x * x, y * y, z * z, w * w};
            *reinterpret_cast<PcQuad *>(s + e) = q;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
#endif
