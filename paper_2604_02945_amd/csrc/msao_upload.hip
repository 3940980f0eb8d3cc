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
// stream (which is a barrier packet of its own). A call that is being recorded
// into a graph takes no slot: the graph's replays come whenever they like, and
// would find other tables there.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "msao_internal.h"
#include "msao_upload.h"

namespace msao {
namespace {

__global__ __launch_bounds__(kUploadBlock) void k_upload(UploadArgs a)
{
    upload_tables<int64_t>(a, a.src);
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
    upload_tables<int>(u.a, (const uint8_t*)(kernel_args() + offsetof(UploadInline, tables)));
}

// One block per piece: 3,840 bytes are 240 threads' 16 bytes.
__global__ __launch_bounds__(kUploadBlock) void k_upload_piece(UploadPiece u)
{
    static_assert(kUploadPiece <= 16 * kUploadBlock, "one 16-byte chunk a thread");
    const uvec4* src = (const uvec4*)(const uint8_t*)(kernel_args() + offsetof(UploadPiece, tables));
    if (threadIdx.x * 16u < u.bytes) ((uvec4*)u.dst)[threadIdx.x] = src[threadIdx.x];
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

int launch_upload_pieces(const UploadArgs& a, int blocks, void* stream)
{
    if (blocks < 1 || blocks > kUploadMaxBlocks || a.copy_bytes % 16 != 0 || !a.src || !a.dst) return (int)hipErrorInvalidValue;
    for (uint64_t at = 0; at < a.copy_bytes; at += kUploadPiece) {
        UploadPiece u;
        u.dst = a.dst + at;
        u.bytes = a.copy_bytes - at < kUploadPiece ? (uint32_t)(a.copy_bytes - at) : kUploadPiece;
        memcpy(u.tables, a.src + at, u.bytes);
        hipLaunchKernelGGL(k_upload_piece, dim3(1), dim3(kUploadBlock), 0, (hipStream_t)stream, u);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return (int)e;
    }
    UploadArgs fill = a;  // the segment records now lead the workspace
    fill.src = a.dst;
    fill.copy_units = 0;
    fill.done = nullptr;
    hipLaunchKernelGGL(k_upload, dim3((unsigned)blocks), dim3(kUploadBlock), 0, (hipStream_t)stream, fill);
    return (int)hipGetLastError();
}

}  // namespace msao
