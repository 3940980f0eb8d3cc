// msao_entropy.hip -- gfx950 (CDNA4) kernel for the draft model's confidence
// in MSAO's speculative decoding (Sec. 4.2): per row of draft logits, the
// entropy of its softmax (Eq. 9), the greedy draft token (arg max) and the
// speculation test against the confidence threshold (Eq. 10).
//
// HBM-bound streaming reduction, one pass over the logits: one workgroup per
// row, each lane reading 16-byte chunks with nontemporal buffer loads, the
// next two batches in flight while the current one is reduced. A lane keeps a
// running maximum m, s = sum exp(x - m) and t = sum exp(x - m)(x - m) over its
// chunks, so that H = ln s - t / s needs no second pass and no cancellation
// against m. Per batch of chunks the batch maximum is taken first; only when
// it exceeds m are s and t rescaled (and the arg max searched), which after
// the first batches is rare. Lane states merge by shuffles, then across the
// block's wavefronts through LDS.
//
// With a few rows (a decode step) one workgroup per row is bound by one CU's
// latency, so a row is cut into up to 64 parts of at least one batch (16 KiB):
// each workgroup leaves its state in a slot of device memory and the last to
// arrive at a row merges them. Nothing waits on the device. A call that gets no
// slot takes one workgroup of 1,024 threads per row, whose four groups take the
// same parts in turn and whose states merge in the same order: the results of a
// call do not depend, in any bit, on what else is in flight.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "msao_internal.h"

namespace msao {
namespace {

constexpr int kEntWave = 64;
constexpr float kLog2e = 1.4426950408889634f;
// exp(-200) is far below the smallest normal float: clamping the difference
// that multiplies exp(x - m) in t only matters for x = -inf, whose term is
// then 0 * -200 = 0 instead of 0 * -inf = NaN. A NaN logit still makes s NaN.
constexpr float kMinDiff = -200.0f;
// A maximum whose product with log2(e) is no finite float (a row, or what has
// been seen of it, masked with the type's lowest value).
constexpr float kFarMax = 2.3e38f;
// Difference of two maxima in log2 units, at least what makes 2^dm 0: a difference
// that overflows would turn the product with the sums into 0 * inf.
__device__ __forceinline__ float max_diff(float lower, float upper) { return fmaxf((lower - upper) * kLog2e, -1000.0f); }

typedef unsigned int ent_vec4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t ent_rsrc_t;

__device__ __forceinline__ ent_rsrc_t ent_rsrc(const void* base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, 0x00020000);
}

// nontemporal: every logit is read once
__device__ __forceinline__ ent_vec4 ent_load(ent_rsrc_t r, int off)
{
    return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 2);
}

// Softmax statistics of a set of logits: maximum m (first index idx),
// s = sum 2^(L (x - m)) = sum exp(x - m) and u = sum 2^(L (x - m)) L (x - m)
// with L = log2(e), i.e. u = L t for t = sum exp(x - m) (x - m). Keeping u in
// log2 units lets one fma give the exponent: L x - L m.
struct Acc {
    float m, s, u;
    int idx;
};

// Merge b into a: the larger maximum wins (the lower index on equal maxima)
// and the other side's sums are rescaled to it. Only an empty side (s == 0)
// is skipped, so a NaN sum still reaches the result.
__device__ __forceinline__ Acc acc_merge(Acc a, Acc b)
{
    if (b.m > a.m || (b.m == a.m && b.idx < a.idx)) {
        const Acc c = a;
        a = b;
        b = c;
    }
    if (b.s != 0.0f) {
        const float dm = max_diff(b.m, a.m);
        const float sc = __builtin_amdgcn_exp2f(dm);
        a.u = fmaf(fmaf(dm, b.s, b.u), sc, a.u);
        a.s = fmaf(b.s, sc, a.s);
    }
    return a;
}

// The lane's value with DPP control CTRL in the rows of ROWS, `old` where there is none.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_i(int old, int v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xF, false);
}

// op over the wavefront, in every lane: four shifts within each row of 16 lanes, then
// lane 15 of a row to the next row and lane 31 to the upper half. id: op(x, id) = x.
template <typename Op>
__device__ __forceinline__ int wave_reduce(int v, int id, Op op)
{
    v = op(v, dpp_i<0x111, 0xF>(id, v));
    v = op(v, dpp_i<0x112, 0xF>(id, v));
    v = op(v, dpp_i<0x114, 0xF>(id, v));
    v = op(v, dpp_i<0x118, 0xF>(id, v));
    v = op(v, dpp_i<0x142, 0xA>(id, v));
    v = op(v, dpp_i<0x143, 0xC>(id, v));
    return __builtin_amdgcn_readlane(v, kEntWave - 1);
}

__device__ __forceinline__ float wave_sum(float v)
{
    return __int_as_float(wave_reduce(__float_as_int(v), 0, [](int a, int b) {
        return __float_as_int(__int_as_float(a) + __int_as_float(b));
    }));
}

// The lanes' states merged, in every lane: their maximum first, so that each
// lane rescales its sums once.
__device__ __forceinline__ Acc wave_merge(const Acc& a)
{
    Acc r;
    r.m = __int_as_float(wave_reduce(__float_as_int(a.m), (int)0xFF800000u, [](int x, int y) {
        return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y)));
    }));
    r.idx = wave_reduce(a.m == r.m ? a.idx : 0x7FFFFFFF, 0x7FFFFFFF, [](int x, int y) { return x < y ? x : y; });
    const float dm = max_diff(a.m, r.m);  // (a lane without a finite value stays at 0)
    const float sc = __builtin_amdgcn_exp2f(dm);
    r.s = wave_sum(a.s * sc);
    r.u = wave_sum(fmaf(dm, a.s, a.u) * sc);
    return r;
}

// The state of no logits: never the lower index.
constexpr Acc kEmpty{-__builtin_huge_valf(), 0.0f, 0.0f, 0x7FFFFFFF};

template <int DT> struct EntLane;
template <> struct EntLane<kBF16> {
    static constexpr int EPC = 8;  // elements per 16-byte chunk
    __device__ static __forceinline__ void widen(const ent_vec4& v, float* x)
    {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            x[2 * w] = __uint_as_float(v[w] << 16);
            x[2 * w + 1] = __uint_as_float(v[w] & 0xFFFF0000u);
        }
    }
    __device__ static __forceinline__ float element(const uint8_t* row, int64_t i)
    {
        return __uint_as_float((uint32_t)((const uint16_t*)row)[i] << 16);
    }
};
template <> struct EntLane<kF32> {
    static constexpr int EPC = 4;
    __device__ static __forceinline__ void widen(const ent_vec4& v, float* x)
    {
#pragma unroll
        for (int w = 0; w < 4; ++w) x[w] = __uint_as_float(v[w]);
    }
    __device__ static __forceinline__ float element(const uint8_t* row, int64_t i)
    {
        return ((const float*)row)[i];
    }
};

// Add the N values x to the lane state; x[j] is element first + stride_of(j)
// (index(j) gives it), used only when the maximum moves.
template <int N, typename IndexOf>
__device__ __forceinline__ void acc_add(Acc& a, const float (&x)[N], IndexOf index)
{
    float cm = x[0];
#pragma unroll
    for (int j = 1; j < N; ++j) cm = fmaxf(cm, x[j]);
    if (cm > a.m) {
        // position of the first maximum, then its index (one computation)
        int js = 0;
#pragma unroll
        for (int j = N - 1; j >= 0; --j)
            if (x[j] == cm) js = j;
        const int at = index(js);
        if (a.s > 0.0f) {
            const float dm = max_diff(a.m, cm);
            const float sc = __builtin_amdgcn_exp2f(dm);
            a.u = fmaf(dm, a.s, a.u) * sc;
            a.s *= sc;
        }
        a.m = cm;
        a.idx = at;
    }
    // While nothing finite has been seen (m = -inf) the values are -inf (they
    // contribute 0) or NaN (which must reach s): take the exponent against 0,
    // since -inf - (-inf) would turn every -inf into NaN.
    const float nml = a.m == -INFINITY ? 0.0f : -a.m * kLog2e;
    // A -inf logit gives e = 0 and d = -inf, whose product must be 0, not
    // NaN. The sums are taken without a clamp on d; a -inf then shows as a
    // NaN u beside a finite s (a NaN logit makes s NaN too), and only then is
    // u summed again with d clamped, from the values still in registers (the
    // same for the lowest value beside ordinary ones). Where the maximum itself is
    // so far from 0 that L m overflows, both sums are taken again from L (x - m).
    // Both ways give the same bits wherever none of that occurs.
    float s = a.s, u = a.u;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const float d = fmaf(x[j], kLog2e, nml);  // L (x - m)
        const float e = __builtin_amdgcn_exp2f(d);
        s += e;
        u = fmaf(e, d, u);
    }
    const bool far = fabsf(a.m) > kFarMax && a.m != -INFINITY;
    if (__ballot((__builtin_isnan(u) && !__builtin_isnan(s)) || far) != 0) {
        s = a.s;
        u = a.u;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float d = far ? (x[j] - a.m) * kLog2e : fmaf(x[j], kLog2e, nml);
            const float e = __builtin_amdgcn_exp2f(d);
            s += e;
            u = fmaf(e, fmaxf(d, kMinDiff * kLog2e), u);
        }
    }
    a.s = s;
    a.u = u;
}

// The state that the row's workgroups merge to, in every lane of the last of
// them to come here; false in the others. Called by one whole wavefront, whose
// lane 0 holds the workgroup's state. The parts are written through to where
// every XCD reads them, and the counters order them.
__device__ __forceinline__ bool meet(const EntArgs& a, int row, int part, Acc& acc)
{
    const int lane = threadIdx.x & (kEntWave - 1);
    EntPart* parts = a.slot->part + row * a.parts;
    uint32_t before = 0;
    if (lane == 0) {
        const uint32_t w[4] = {__float_as_uint(acc.m), __float_as_uint(acc.s), __float_as_uint(acc.u), (uint32_t)acc.idx};
#pragma unroll
        for (int i = 0; i < 4; ++i) __hip_atomic_store(&parts[part].w[i], w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        before = __hip_atomic_fetch_add(&a.slot->row_count[row], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    }
    if ((int)__shfl(before, 0) != a.parts - 1) return false;
    acc = kEmpty;
    if (lane < a.parts) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = __hip_atomic_load(&parts[lane].w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        acc = Acc{__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]), (int)w[3]};
    }
    acc = wave_merge(acc);
    return true;
}

// After the row's parts are read: the counters back to zero, and the slot
// back to the host with the last row.
__device__ __forceinline__ void leave(const EntArgs& a, int row)
{
    __hip_atomic_store(&a.slot->row_count[row], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t before = __hip_atomic_fetch_add(&a.slot->rows_done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (before != (uint32_t)a.rows - 1u) return;
    __hip_atomic_store(&a.slot->rows_done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.done, a.ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// How a row is spread: one workgroup; one workgroup per part; one workgroup
// whose kEntGroups groups of kEntBlock threads take the parts in turn.
enum EntMode { kWhole, kSplit, kGrouped };
constexpr int kEntWaves = kEntBlock / kEntWave;

// This thread's state over chunks [c_lo, c_lo + nfull) of the row at `row`,
// and over the elements past the row's last whole chunk if they follow.
template <int DT, int U>
__device__ __forceinline__ Acc part_state(const EntArgs& a, const uint8_t* row, int c_lo, int per, int tid)
{
    using L = EntLane<DT>;
    constexpr int EPC = L::EPC;
    constexpr int STEP = U * kEntBlock;  // chunks per batch of the block
    const int e_lo = c_lo * EPC;                         // the part's first element
    const uint8_t* base = row + (int64_t)c_lo * 16;
    const int row_chunks = a.vocab / EPC;                // whole 16-byte chunks of the row
    const int nfull = min(per, row_chunks - c_lo);       // and of the part
    const int npair = nfull / (2 * STEP) * (2 * STEP);  // chunks of whole pairs of batches
    const ent_rsrc_t rs = ent_rsrc(base, nfull * 16);
    Acc acc{-INFINITY, 0.0f, 0.0f, 0};
    float x[U * EPC];
    // batches in two register sets used in turn: once a batch is widened its
    // set loads the batch after next, so two batches are in flight while one
    // is reduced. The loads are unconditional, so that no register set needs
    // a copy and the loop has one way back to its head (whose wait is then for
    // the first set only): past the row they fall outside the buffer
    // resource, read nothing and return zeros (the offsets stay below 2^31: a
    // row is at most 2^31 - 2^20 bytes).
    ent_vec4 ba[U], bb[U];
    auto load = [&](ent_vec4 (&b)[U], int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = ent_load(rs, (c0 + u * kEntBlock + tid) * 16);
    };
    auto reduce = [&](int c0) {
        acc_add<U * EPC>(acc, x, [&](int j) { return e_lo + (c0 + (j / EPC) * kEntBlock + tid) * EPC + j % EPC; });
    };
    // widen a set whose chunks may pass the row's last whole chunk: those read as -inf
    auto widen_masked = [&](const ent_vec4 (&b)[U], int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            L::widen(b[u], &x[u * EPC]);
            if (c0 + u * kEntBlock + tid >= nfull) {
#pragma unroll
                for (int j = 0; j < EPC; ++j) x[u * EPC + j] = -INFINITY;
            }
        }
    };
    load(ba, 0);
    // all of the first set's loads are issued before the second set's
    __builtin_amdgcn_sched_barrier(0);
    load(bb, STEP);
    for (int c0 = 0; c0 < npair; c0 += 2 * STEP) {
#pragma unroll
        for (int u = 0; u < U; ++u) L::widen(ba[u], &x[u * EPC]);
        load(ba, c0 + 2 * STEP);
        reduce(c0);
#pragma unroll
        for (int u = 0; u < U; ++u) L::widen(bb[u], &x[u * EPC]);
        load(bb, c0 + 3 * STEP);
        reduce(c0 + STEP);
    }
    // the rest of the whole chunks, fewer than two batches, already loaded
    if (npair < nfull) {
        widen_masked(ba, npair);
        reduce(npair);
    }
    if (npair + STEP < nfull) {
        widen_masked(bb, npair + STEP);
        reduce(npair + STEP);
    }
    // the elements past the last whole chunk, one per thread
    const int tail = c_lo + nfull == row_chunks ? a.vocab - row_chunks * EPC : 0;
    if (tid < tail) {
        const int i = nfull * EPC + tid;
        float x1[1] = {L::element(base, i)};
        acc_add<1>(acc, x1, [&](int) { return e_lo + i; });
    }
    return acc;
}

// The states of the row's parts (whole batches each), wavefront by wavefront as
// part_state and wave_merge give them, by a workgroup of kEntGroups groups. The
// batches of a group follow one another over its parts; each is loaded while the
// one before it is reduced, and the groups share the CU's SIMDs.
template <int DT, int U>
__device__ __forceinline__ void grouped_states(const EntArgs& a, const uint8_t* row, Acc (*part_acc)[kEntWaves])
{
    using L = EntLane<DT>;
    constexpr int EPC = L::EPC;
    constexpr int STEP = U * kEntBlock;
    const int group = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kEntBlock);
    const int tid = threadIdx.x & (kEntBlock - 1), lane = tid & (kEntWave - 1), wid = tid >> 6;
    const int row_chunks = a.vocab / EPC;
    const ent_rsrc_t rs = ent_rsrc(row, row_chunks * 16);
    float x[U * EPC];
    ent_vec4 b[U];
    auto load = [&](int c0) {  // (past the row: zeros; the offsets stay below 2^31, as there)
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = ent_load(rs, (c0 + u * kEntBlock + tid) * 16);
    };
    Acc acc{-INFINITY, 0.0f, 0.0f, 0};
    int p = group, c = 0;
    if (p < a.parts) load(p * a.per);
    while (p < a.parts) {
        const int c0 = p * a.per + c, end = min((p + 1) * a.per, row_chunks);  // every part has a chunk
#pragma unroll
        for (int u = 0; u < U; ++u) {
            L::widen(b[u], &x[u * EPC]);
            if (c0 + STEP > row_chunks && c0 + u * kEntBlock + tid >= row_chunks) {
#pragma unroll
                for (int j = 0; j < EPC; ++j) x[u * EPC + j] = -INFINITY;
            }
        }
        const bool last = c0 + STEP >= end;  // of the part
        const int np = last ? p + kEntGroups : p, nc = last ? 0 : c + STEP;
        if (np < a.parts) load(np * a.per + nc);
        acc_add<U * EPC>(acc, x, [&](int j) { return (c0 + (j / EPC) * kEntBlock + tid) * EPC + j % EPC; });
        if (last) {
            // the elements past the last whole chunk, one per thread
            const int i = row_chunks * EPC + tid;
            if (p == a.parts - 1 && i < a.vocab) {
                float x1[1] = {L::element(row, i)};
                acc_add<1>(acc, x1, [&](int) { return i; });
            }
            acc = wave_merge(acc);
            if (lane == 0) part_acc[p][wid] = acc;
            acc = Acc{-INFINITY, 0.0f, 0.0f, 0};
        }
        p = np;
        c = nc;
    }
}

__device__ __forceinline__ Acc merge_waves(const Acc (&w)[kEntWaves])
{
    Acc r = w[0];
#pragma unroll
    for (int i = 1; i < kEntWaves; ++i) r = acc_merge(r, w[i]);
    return r;
}

template <int DT, int U, EntMode MODE>
__global__ __launch_bounds__(MODE == kGrouped ? kEntGroups * kEntBlock : kEntBlock) void k_entropy(EntArgs a)
{
    const int row = MODE == kSplit ? (int)blockIdx.x / a.parts : (int)blockIdx.x;
    const int part = MODE == kSplit ? (int)blockIdx.x - row * a.parts : 0;
    const int lane = threadIdx.x & (kEntWave - 1);
    const uint8_t* base = a.logits + (int64_t)row * a.row_bytes;
    Acc r;
    if constexpr (MODE == kGrouped) {
        __shared__ Acc part_acc[kEntSplitBlocks][kEntWaves];
        grouped_states<DT, U>(a, base, part_acc);
        __syncthreads();
        if (threadIdx.x >= kEntWave) return;
        r = wave_merge(lane < a.parts ? merge_waves(part_acc[lane]) : kEmpty);
        if (lane != 0) return;
    } else {
        __shared__ Acc wave_acc[kEntWaves];
        const int tid = threadIdx.x;
        const Acc acc = wave_merge(part_state<DT, U>(a, base, part * a.per, a.per, tid));
        if (lane == 0) wave_acc[tid >> 6] = acc;
        __syncthreads();
        if (tid >= (MODE == kSplit ? kEntWave : 1)) return;
        r = merge_waves(wave_acc);
        if constexpr (MODE == kSplit) {
            if (!meet(a, row, part, r)) return;
            if (tid != 0) return;
            leave(a, row);
        }
    }
    // Eq. 9: H = -sum p ln p = ln s - t / s with p = exp(x - m) / s and t = u / L
    const float H = __logf(r.s) - (r.u * 0.6931471805599453f) / r.s;
    const float Hn = H * a.inv_log_vocab;
    if (a.entropy) a.entropy[row] = H;
    if (a.entropy_norm) a.entropy_norm[row] = Hn;
    if (a.draft_token) a.draft_token[row] = r.idx;
    if (a.speculate) a.speculate[row] = Hn <= a.theta ? 1 : 0;  // Eq. 10
}

template <int DT, EntMode MODE>
void enqueue(const EntArgs& a, hipStream_t st, void* ev0, void* ev1)
{
    const dim3 grid((unsigned)a.rows * (unsigned)(MODE == kSplit ? a.parts : 1)),
        block(MODE == kGrouped ? kEntGroups * kEntBlock : kEntBlock);
    if (ev0 && ev1)
        hipExtLaunchKernelGGL((k_entropy<DT, kEntUnits, MODE>), grid, block, 0, st, (hipEvent_t)ev0, (hipEvent_t)ev1, 0, a);
    else
        hipLaunchKernelGGL((k_entropy<DT, kEntUnits, MODE>), grid, block, 0, st, a);
}

template <int DT>
void enqueue_any(const EntArgs& a, hipStream_t st, void* ev0, void* ev1)
{
    if (a.parts == 1) enqueue<DT, kWhole>(a, st, ev0, ev1);
    else if (a.slot) enqueue<DT, kSplit>(a, st, ev0, ev1);
    else enqueue<DT, kGrouped>(a, st, ev0, ev1);
}

std::mutex g_slot_mu;
uint64_t g_slot_taken[kMaxScratchDevices] = {};
static_assert(kEntDeviceSlots <= 64, "a bit each");

}  // namespace

static __device__ __align__(256) EntSlot slots[kEntDeviceSlots];  // zero when the code object is loaded

int ent_slots_take(int device, int want, EntSlot** out)
{
    if (device < 0 || device >= kMaxScratchDevices) return 0;
    std::lock_guard<std::mutex> lock(g_slot_mu);
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(slots)) != hipSuccess || !p) {
        (void)hipGetLastError();
        return 0;
    }
    int n = 0;
    for (int i = 0; i < kEntDeviceSlots && n < want; ++i)
        if (!(g_slot_taken[device] >> i & 1)) {
            g_slot_taken[device] |= 1ull << i;
            out[n++] = (EntSlot*)p + i;
        }
    return n;
}

void ent_slots_give(int device, int n, EntSlot* const* given)
{
    if (n <= 0) return;
    std::lock_guard<std::mutex> lock(g_slot_mu);
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(slots)) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    for (int i = 0; i < n; ++i)
        if (given[i]) g_slot_taken[device] &= ~(1ull << (given[i] - (EntSlot*)p));
}

// Parts per row that a call of these sizes is worth. A workgroup takes 0.4 us a
// batch (fp32; 0.8 bf16) and 3 us besides; the meeting of a row's workgroups adds
// 2 us and about 0.05 us for every one, whose release writes back an L2. So the
// parts are 64 in all, and rows that take a workgroup less than 9 us or so (16
// batches of fp32, 12 of bf16) are not cut: 65,536 fp32 logits 10.4 -> 5.7 us, but
// 32,000 5.5 -> 6.1. Of 151,936 logits, one row of fp32 18.7 -> 5.6 us and of bf16
// 18.4 -> 6.1, 16 rows 19.3 -> 10.3 and 19.4 -> 9.8; with up to 1,024 workgroups 16
// rows took 16.7 and 64 rows 22.6 against 19.8. Without a slot (a call recorded into a
// graph, launch to launch) 19.1 -> 18.1 and 18.3 -> 14.4, 16 rows 19.9 -> 14.2 and
// 19.9 -> 13.3.
void ent_split(int64_t rows, int64_t vocab, int dtype, int* parts, int* per)
{
    const int64_t chunks = vocab / (dtype == kBF16 ? 8 : 4), batch = (int64_t)kEntUnits * kEntBlock;
    int64_t p = 1;
    if (rows <= kEntSplitRows && chunks >= (dtype == kBF16 ? kEntSplitBatchesBF16 : kEntSplitBatchesF32) * batch)
        p = std::min<int64_t>(kEntSplitBlocks / rows, (chunks + batch - 1) / batch);
    *parts = 1;
    *per = (int)chunks;
    if (p < 2) return;
    const int64_t c = ((chunks + p - 1) / p + batch - 1) / batch * batch;  // whole batches: a part of one takes a batch's time
    *per = (int)c;
    *parts = (int)((chunks + c - 1) / c);  // every part has a chunk
}

int launch_entropy(const EntArgs& a, void* stream, void* ev0, void* ev1)
{
    if (a.rows <= 0) return kNoLaunch;
    const hipStream_t st = (hipStream_t)stream;
    if (a.parts < 1 || (a.parts > 1 && (a.rows > kEntSplitRows || (int64_t)a.rows * a.parts > kEntSplitBlocks)) ||
        (a.slot && !a.done))
        return (int)hipErrorInvalidValue;
    if (a.dtype == kBF16) enqueue_any<kBF16>(a, st, ev0, ev1);
    else enqueue_any<kF32>(a, st, ev0, ev1);
    return (int)hipGetLastError();
}

}  // namespace msao
