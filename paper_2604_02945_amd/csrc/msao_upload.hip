// msao_upload.hip -- brings a call's tables from the context's pinned staging
// into the workspace.
//
// Bound by latency: one read of host memory over the host link (about 2 us),
// then a few KB to a few hundred KB of stores. One kernel on the caller's
// stream does it, in place of a copy command: a copy of more than a few KB
// goes to a DMA engine, whose hand-over from and to the compute queue, with
// the event that guarded the staging slot, left the GPU idle for 22-28 us
// before the scoring pass (a small copy, done by a blit kernel, for 24 us
// around its 2 us); this kernel and the gaps around it take about 5 us. The
// "segment of each item" arrays, most of the bytes (200 KB of 230 on a batch
// of 32 tri-modal requests), are runs of one value, so they are not staged:
// the kernel writes them from the segment records.
//
// Each block that has read the staging slot says so with its own word in
// host memory, so that the host can reuse the slot without an event on the
// stream (which is a barrier packet of its own).
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "msao_internal.h"

namespace msao {
namespace {

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

// The tables of `a`, staged at src.
__device__ __forceinline__ void upload_tables(const UploadArgs& a, const uint8_t* staged)
{
    const int units = a.copy_units + a.n * a.fill_parts;
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        if (u < a.copy_units) {
            // 16-byte pieces (the staged bytes and both addresses are multiples of 16)
            constexpr int V = kUploadCopyBytes / (16 * kUploadBlock);
            const uvec4* src = (const uvec4*)staged;
            uvec4* dst = (uvec4*)a.dst;
            const uint32_t pieces = a.copy_bytes / 16u;
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
        const int f = u - a.copy_units, s = f / a.fill_parts, part = f - s * a.fill_parts;
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

__global__ __launch_bounds__(kUploadBlock) void k_upload(UploadArgs a)
{
    upload_tables(a, a.src);
    if (a.done) {
        // every thread's reads of the slot have returned (its stores took their
        // values), and nothing that it wrote need be visible to the host
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(a.done + blockIdx.x, a.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Tables of at most kUploadInline bytes travel in the kernel's arguments,
// which the launch brings to the device anyway: no read over the host link, no
// staging slot, and a graph holds its own copy. For one image request 5.0 ->
// 2.9 us in the trace; 3 KiB (a dozen segments) is what leaves room for the
// other arguments in the 4 KiB that a launch takes.
__global__ __launch_bounds__(kUploadBlock) void k_upload_inline(UploadInline u)
{
    // by address, since the members of a by-value argument cannot be indexed in place
    const __attribute__((address_space(4))) uint8_t* args =
        (const __attribute__((address_space(4))) uint8_t*)__builtin_amdgcn_kernarg_segment_ptr();
    upload_tables(u.a, (const uint8_t*)(args + offsetof(UploadInline, tables)));
}

}  // namespace

int launch_upload(const UploadArgs& a, int blocks, void* stream)
{
    if (blocks < 1 || blocks > kUploadMaxBlocks || a.copy_bytes % 16 != 0 || !a.src || !a.dst) return (int)hipErrorInvalidValue;
    if (a.copy_bytes <= kUploadInline) {
        UploadInline u;
        u.a = a;
        memcpy(u.tables, a.src, a.copy_bytes);
        hipLaunchKernelGGL(k_upload_inline, dim3((unsigned)blocks), dim3(kUploadBlock), 0, (hipStream_t)stream, u);
        return (int)hipGetLastError();
    }
    hipLaunchKernelGGL(k_upload, dim3((unsigned)blocks), dim3(kUploadBlock), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

}  // namespace msao
