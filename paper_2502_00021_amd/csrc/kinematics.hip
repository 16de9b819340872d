// Producer stage of libpxr: joint angles -> rigid-body poses on the device, so
// that the renderer's input never has to come from the host (PixelBrax, arXiv
// 2502.00021, section 1: the whole loop, environment step included, stays on
// the accelerator).  gfx950 only.
//
// A workgroup of four wavefronts takes 64 frames, one per lane, and shares out their bodies: the skeleton's
// records come in order of depth (free bodies, then their children, ...), a depth's bodies are dealt to the four
// wavefronts, and a barrier separates the depths.  What does not depend on the parent - the free poses, sine and
// cosine of every half angle - is done for all bodies at once before the first of them.  What bounds the stage is
// latency, not work: a frame is a chain of dependent quaternion products, and its length here is the tree's depth
// (4 for a humanoid of 15 bodies) instead of its number of bodies.  Measured on that
// skeleton against one wavefront that walked all bodies of its 64 frames with staged inputs: 30 frames 12.0 -> 4.5 us
// (an empty-handed launch takes 4), 196 608 frames 50.7 -> 21.1 us = 4.9 TB/s, what a large copy reaches; the 7-link
// chain, whose depth is its length, 8.8 -> 4.8 us for 256 frames.
// The records are wave-uniform and arrive through scalar loads, a depth's first one before the barrier that opens
// it.  Angles and free poses are read from memory as each lane needs them (a workgroup's are a contiguous few KB:
// every line is fetched once).  The poses of the 64 frames live in LDS as the image of the output chunk they become,
// one row of 7 K floats per frame; an even row gets one float of padding, so that the row stride is odd and the
// lanes of a wavefront, one row each, use different banks.

#include <hip/hip_runtime.h>

#include "hinge.h"
#include "pxr_internal.h"

namespace pxr {
namespace {

constexpr uint32_t kFkFrames = 64;    // frames per workgroup: one per lane of a wavefront
constexpr uint32_t kFkWaves = 4;      // wavefronts that share the frames' bodies
constexpr uint32_t kFkThreads = kFkFrames * kFkWaves;
constexpr uint32_t kFkAhead = 4;      // bodies a wavefront has requests in flight for before the first depth

__global__ __launch_bounds__(kFkThreads) void fk_kernel(const SkeletonConsts sk, const float* __restrict__ free_poses,
                                                        const float* __restrict__ angles, uint32_t n_frames,
                                                        float* __restrict__ poses) {
    extern __shared__ __align__(16) unsigned char lds[];
    float* pose = reinterpret_cast<float*>(lds);  // [kFkFrames][stride]
    const uint32_t n_row = sk.K * 7u, stride = n_row | 1u;

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t f0 = blockIdx.x * kFkFrames;               // first frame of this workgroup
    const uint32_t nf = min(kFkFrames, n_frames - f0);        // frames it holds (ragged tail)
    float* row = pose + lane * stride;

    // ---- what depends on no parent, all bodies at once (lanes past the last frame repeat it and are not stored)
    {
        const size_t frame = f0 + min(lane, nf - 1u);
        const float* my_angles = angles + frame * sk.J;
        const float* my_free = free_poses + frame * (sk.F * 7u);
        for (uint32_t i0 = wave; i0 < sk.K; i0 += kFkWaves * kFkAhead) {
            float theta[kFkAhead];
#pragma unroll
            for (uint32_t u = 0; u < kFkAhead; ++u) {
                const uint32_t i = min(i0 + u * kFkWaves, sk.K - 1u);
                const SkeletonRecord& t = sk.records[i];
                theta[u] = 0.0f;
                if (t.parent >= 0 && t.slot >= 0) theta[u] = my_angles[t.slot];
            }
#pragma unroll
            for (uint32_t u = 0; u < kFkAhead; ++u) {
                const uint32_t i = i0 + u * kFkWaves;
                if (i >= sk.K) break;
                const SkeletonRecord& t = sk.records[i];
                float* o = row + t.body * 7u;
                if (t.parent < 0) {
                    const float* src = my_free + t.slot * 7;
                    float v[7];
#pragma unroll
                    for (int c = 0; c < 7; ++c) v[c] = src[c];
#pragma unroll
                    for (int c = 0; c < 7; ++c) o[c] = v[c];
                } else {
                    sincos_half(theta[u], o[4], o[3]);
                }
            }
        }
    }

    // ---- the tree, depth by depth
    uint32_t begin = sk.depth_begin[1];
    for (uint32_t d = 1; d < sk.depths; ++d) {
        const uint32_t end = sk.depth_begin[d + 1];
        uint32_t i = begin + wave;
        SkeletonRecord t = sk.records[min(i, sk.K - 1u)];
        __syncthreads();
        while (i < end) {
            float* o = row + t.body * 7u;
            hinge_pose(t, row + t.parent * 7, o[3], o[4], o);  // (cosine and sine were left there for all bodies before the first depth)
            i += kFkWaves;
            if (i < end) t = sk.records[i];
        }
        begin = end;
    }
    __syncthreads();

    // ---- the workgroup's contiguous output chunk
    const uint32_t n_o = nf * n_row;
    float* dst = poses + (size_t)f0 * n_row;
    if (stride == n_row && (reinterpret_cast<uintptr_t>(poses) & 15u) == 0u) {
        // (no padding: LDS holds the chunk as it is.  A chunk starts 64 rows, a multiple of 16 bytes, after another.)
        const uint32_t n_quads = n_o >> 2;
        for (uint32_t i = threadIdx.x; i < n_quads; i += kFkThreads)
            reinterpret_cast<float4*>(dst)[i] = reinterpret_cast<const float4*>(pose)[i];
        const uint32_t i = (n_quads << 2) + threadIdx.x;
        if (i < n_o) dst[i] = pose[i];
    } else {
        const uint32_t pad = stride - n_row;
        const uint32_t magic = 0xFFFFFFFFu / n_row + 1u;  // (i / n_row by multiplication: i < 64 * n_row, rows of 7 floats and more)
#pragma unroll 4
        for (uint32_t i = threadIdx.x; i < n_o; i += kFkThreads) dst[i] = pose[i + pad * __umulhi(i, magic)];
    }
}

}  // namespace

uint32_t fk_lds_bytes(const SkeletonConsts& sk) { return kFkFrames * (sk.K * 7u | 1u) * 4u; }

int prepare_fk_kernel(std::string& err) {
    const hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(&fk_kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (rc != hipSuccess) {
        err = std::string("hipFuncSetAttribute(MaxDynamicSharedMemorySize) failed: ") + hipGetErrorString(rc);
        return PXR_ERR_DEVICE;
    }
    return PXR_OK;
}

int launch_fk(const SkeletonConsts& sk, const float* d_free_poses, const float* d_angles, uint32_t n_frames,
              float* d_poses, void* stream, std::string& err) {
    const uint32_t blocks = (n_frames + kFkFrames - 1) / kFkFrames;
    hipLaunchKernelGGL(fk_kernel, dim3(blocks), dim3(kFkThreads), fk_lds_bytes(sk), reinterpret_cast<hipStream_t>(stream), sk,
                       d_free_poses, d_angles, n_frames, d_poses);
    const hipError_t rc = hipGetLastError();
    if (rc != hipSuccess) {
        err = std::string("kernel launch failed: ") + hipGetErrorString(rc);
        return PXR_ERR_DEVICE;
    }
    return PXR_OK;
}

}  // namespace pxr
