// msao_upload.h -- what the upload kernel does with a call's tables, for the
// kernels that bring them along themselves.
#ifndef MSAO_UPLOAD_H
#define MSAO_UPLOAD_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msao_internal.h"

namespace msao {
namespace {

// The arguments of the running kernel, to be read by address: the members of
// an argument passed by value cannot be indexed in place.
typedef const __attribute__((address_space(4))) uint8_t* args_ptr;
__device__ __forceinline__ args_ptr kernel_args() { return (args_ptr)__builtin_amdgcn_kernarg_segment_ptr(); }

typedef unsigned int uvec4 __attribute__((ext_vector_type(4)));

// Entries [begin, begin + count) of an array take the value s; of them this
// unit writes the stripes part, part + parts, ... of kUploadFill entries.
__device__ __forceinline__ void fill_run(int32_t* dst, int begin, int count, int s, int part, int parts)
{
    for (int i0 = part * kUploadFill; i0 < count; i0 += parts * kUploadFill) {
        const int i1 = min(count, i0 + kUploadFill);
        for (int i = i0 + (int)threadIdx.x; i < i1; i += kUploadBlock) dst[begin + i] = s;
    }
}

// The tables of `a`, staged at src. Unit: of the units' indices (int for tables of
// at most kUploadInline bytes, a dozen segments).
template <typename Unit>
__device__ __forceinline__ void upload_tables(const UploadArgs& a, const uint8_t* staged)
{
    const Unit units = a.copy_units + (Unit)a.n * a.fill_parts;
    for (Unit u = blockIdx.x; u < units; u += gridDim.x) {
        if (u < a.copy_units) {
            // 16-byte pieces (the staged bytes and both addresses are multiples of 16)
            constexpr int V = kUploadCopyBytes / (16 * kUploadBlock);
            const uvec4* src = (const uvec4*)staged;
            uvec4* dst = (uvec4*)a.dst;
            const uint32_t pieces = (uint32_t)(a.copy_bytes / 16u);
            const uint32_t p0 = (uint32_t)u * (kUploadCopyBytes / 16) + threadIdx.x;
            uvec4 v[V];
#pragma unroll
            for (int q = 0; q < V; ++q)
                if (p0 + q * kUploadBlock < pieces) v[q] = src[p0 + q * kUploadBlock];
#pragma unroll
            for (int q = 0; q < V; ++q)
                if (p0 + q * kUploadBlock < pieces) dst[p0 + q * kUploadBlock] = v[q];
            continue;
        }
        const Unit f = u - a.copy_units;
        const int s = a.fill_parts == 1 ? (int)f : (int)(f / a.fill_parts), part = (int)(f - (Unit)s * a.fill_parts);
        const DevSeg& sg = ((const DevSeg*)staged)[s];  // the segment records lead the staged tables
        fill_run(a.wi_seg, sg.wi_begin, sg.n_items, s, part, a.fill_parts);
        fill_run(a.gi_seg, sg.g_begin, sg.n_gather, s, part, a.fill_parts);
        if (sg.head_w) fill_run(a.hb_seg, sg.hb_begin, sg.T, s, part, a.fill_parts);
        if (sg.temporal) fill_run(a.frame_seg, sg.frame_off, sg.T, s, part, a.fill_parts);
        if (sg.fused)
            fill_run(a.cl_seg, sg.cl_begin, (sg.P * sg.ntiles + kClipWaves - 1) / kClipWaves, s, part, a.fill_parts);
        if (a.any_hash)
            fill_run(a.hi_seg, sg.hi_begin, (sg.n_tok + kHashBlockTokens - 1) / kHashBlockTokens, s, part, a.fill_parts);
    }
}

}  // namespace
}  // namespace msao

#endif
