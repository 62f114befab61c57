// The allocation-free entry point: one whole synchronization (the fused kernel,
// or pack, reduce and average, write back where tensors share memory) whose
// device tables and flat bucket buffers live in a file-scope device array instead of memory
// obtained from hipMalloc.  For callers that cannot allocate: code under HIP
// graph capture, tight serving loops, harnesses that forbid allocation.
#include "../../include/ddp_gfx950.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "bucket_plan.h"
#include "ddp_kernels.h"
#include "seg_layout.h"

namespace ddp {
int32_t fail_without_context(int32_t code, const std::string& msg);   // ddp_api.hip
}

namespace {

// Every GPU the library runs on holds its own copy of this array, at its own
// address, until the process ends.  In host code the name below is only a
// handle for hipGetSymbolAddress; the device address is looked up once per
// device (scratch_on) and that pointer is what kernels and fills receive.
static __device__ __align__(256) unsigned char scratch[DDP_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_mu;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (which must be `device`).
hipError_t scratch_on(int device, unsigned char** out) {
    std::lock_guard<std::mutex> lock(g_mu);
    if (g_scratch_ptr[device] == nullptr) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = static_cast<unsigned char*>(p);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

// Host data reaches the device inside kernel arguments: no copy engine, no
// staging buffer, nothing that reads host memory after the call has returned
// (so the call can also be captured into a graph).
constexpr int kPayloadWords = 768;              // 3 KiB per launch
struct Payload { uint32_t w[kPayloadWords]; };

__global__ __launch_bounds__(256) void table_write_kernel(uint32_t* __restrict__ dst, Payload p, int nwords) {
    for (int i = threadIdx.x; i < nwords; i += 256) dst[i] = p.w[i];
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void clear_kernel(u32x4* __restrict__ dst, int64_t nvec) {
    const u32x4 z = {0u, 0u, 0u, 0u};
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < nvec; i += stride) dst[i] = z;
}

hipError_t upload(unsigned char* dst, const void* src, size_t bytes, hipStream_t s) {
    // dst and bytes are multiples of 4 by construction of the layout
    const uint32_t* w = static_cast<const uint32_t*>(src);
    size_t words = bytes / 4;
    uint32_t* d = reinterpret_cast<uint32_t*>(dst);
    while (words > 0) {
        Payload p;
        const int nw = static_cast<int>(words < static_cast<size_t>(kPayloadWords) ? words : kPayloadWords);
        std::memcpy(p.w, w, static_cast<size_t>(nw) * 4);
        hipLaunchKernelGGL(table_write_kernel, dim3(1), dim3(256), 0, s, d, p, nw);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        w += nw; d += nw; words -= static_cast<size_t>(nw);
    }
    return hipSuccess;
}

// Whether no tensor that the call writes (replica 0's) shares a byte with any other tensor it reads.
// Told from the address ranges of whole replicas: each replica's tensors usually come
// from one region, and lists for which that does not hold take the path through the flat buckets.
// Replica 0's own tensors are compared in the order of the list if their addresses ascend or descend in it;
// else they are sorted, up to kSortedTensors of them, where that costs what the flat path's launches
// do (host time of a call with shuffled tensors, R = 2, flat / sorted: 300 49 / 23 us, 2000 171 / 175, 20000
// 1300 / 2046; ascending 20000 flat 1293, sorted 1416, compared in order 1306).
constexpr size_t kSortedTensors = 2000;

struct AddressRange {
    uintptr_t first = UINTPTR_MAX, end = 0;      // empty: end == 0
};

bool writes_are_apart(const ddp::BucketPlan& plan, void* const* grad_ptrs, int32_t R, const uintptr_t* shift) {
    const size_t n = plan.params.size();
    auto bytes_of = [&](size_t i) { return static_cast<uintptr_t>(plan.params[i].numel) * ddp::elem_size(plan.params[i].dtype); };
    AddressRange own;
    bool ascending = true, descending = true;
    uintptr_t before_first = 0, before_end = 0;
    for (size_t i = 0; i < n; ++i) {
        const uintptr_t bytes = bytes_of(i), a = reinterpret_cast<uintptr_t>(grad_ptrs[i]);
        if (bytes == 0) continue;
        if (own.end != 0) {
            ascending = ascending && a >= before_end;
            descending = descending && a + bytes <= before_first;
        }
        before_first = a;
        before_end = a + bytes;
        own.first = std::min(own.first, a);
        own.end = std::max(own.end, a + bytes);
    }
    for (int64_t r = 1; r < R; ++r) {
        void* const* row = grad_ptrs + r * static_cast<int64_t>(n);
        AddressRange other;
        if (shift != nullptr && own.end != 0) other = AddressRange{own.first + shift[r], own.end + shift[r]};
        else for (size_t i = 0; i < n; ++i) {
            const uintptr_t bytes = bytes_of(i), a = reinterpret_cast<uintptr_t>(row[i]);
            if (bytes == 0) continue;
            other.first = std::min(other.first, a);
            other.end = std::max(other.end, a + bytes);
        }
        if (other.first < own.end && own.first < other.end) return false;
    }
    if (ascending || descending) return true;
    if (n > kSortedTensors) return false;
    std::vector<std::pair<uintptr_t, uintptr_t>> sorted;     // replica 0's tensors, [first byte, end)
    sorted.reserve(n);
    for (size_t i = 0; i < n; ++i)
        if (bytes_of(i) != 0) sorted.emplace_back(reinterpret_cast<uintptr_t>(grad_ptrs[i]), reinterpret_cast<uintptr_t>(grad_ptrs[i]) + bytes_of(i));
    std::sort(sorted.begin(), sorted.end());
    for (size_t k = 1; k < sorted.size(); ++k)
        if (sorted[k].first < sorted[k - 1].second) return false;
    return true;
}

// Whether every replica's tensors lie alike (views into one buffer per replica, say): shift[r] = what those of replica r lie
// further on than replica 0's.  Tensors without elements do not count.
bool replicas_alike(const ddp::BucketPlan& plan, void* const* grad_ptrs, int32_t R, uintptr_t* shift, int64_t* base) {
    const int64_t n = static_cast<int64_t>(plan.params.size());
    int64_t b = 0;
    while (b < n && plan.params[b].numel == 0) ++b;
    if (b == n) return false;
    *base = b;
    for (int64_t r = 0; r < R; ++r) {
        void* const* row = grad_ptrs + r * n;
        shift[r] = reinterpret_cast<uintptr_t>(row[b]) - reinterpret_cast<uintptr_t>(grad_ptrs[b]);
        for (int64_t i = b + 1; i < n; ++i)
            if (reinterpret_cast<uintptr_t>(row[i]) != reinterpret_cast<uintptr_t>(grad_ptrs[i]) + shift[r] && plan.params[i].numel != 0) return false;
    }
    return true;
}

#define HIPCHK0(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return ddp::fail_without_context(DDP_ERR_HIP, std::string("ddp_sync_static: ") + #expr + ": " + hipGetErrorString(e_)); \
    } while (0)

}  // namespace

extern "C" int32_t ddp_sync_static(int32_t R, int32_t device, void* stream, int32_t n,
                                   const int64_t* numel, const int32_t* dtype,
                                   void* const* grad_ptrs, uint64_t cap_bytes) {
    using ddp::fail_without_context;
    if (R < 1) return fail_without_context(DDP_ERR_ARG, "ddp_sync_static: R must be at least 1");
    if (R > DDP_MAX_REPLICAS) return fail_without_context(DDP_ERR_UNSUPPORTED, "ddp_sync_static: R above DDP_MAX_REPLICAS");
    if (device < 0 || device >= kMaxDevices) return fail_without_context(DDP_ERR_ARG, "ddp_sync_static: bad device");
    if (n <= 0 || !numel || !dtype || !grad_ptrs)
        return fail_without_context(DDP_ERR_ARG, "ddp_sync_static: n <= 0 or null array");
    ddp::BucketPlan plan;
    plan.params.resize(n);
    for (int32_t i = 0; i < n; ++i) {
        if (numel[i] < 0) return fail_without_context(DDP_ERR_ARG, "ddp_sync_static: negative numel");
        if (dtype[i] != DDP_FP32 && dtype[i] != DDP_FP16 && dtype[i] != DDP_BF16)
            return fail_without_context(DDP_ERR_ARG, "ddp_sync_static: unknown dtype");
        plan.params[i].numel = numel[i];
        plan.params[i].dtype = dtype[i];
    }
    // Sizes first (before any pointer is looked at): a model that cannot fit is refused.
    {
        uint64_t total = 0;
        for (int32_t i = 0; i < n; ++i) {
            const uint64_t b = static_cast<uint64_t>(numel[i]) * static_cast<uint64_t>(ddp::elem_size(dtype[i]));
            if (static_cast<uint64_t>(numel[i]) > (uint64_t(1) << 40) || total + b > (uint64_t(1) << 40)) {
                total = uint64_t(1) << 40;
                break;
            }
            total += b;
        }
        if (total * static_cast<uint64_t>(R + 1) > DDP_STATIC_SCRATCH_BYTES)
            return fail_without_context(DDP_ERR_UNSUPPORTED,
                        "ddp_sync_static: (R + 1) x gradient bytes exceed the static scratch buffer of " +
                        std::to_string(DDP_STATIC_SCRATCH_BYTES) + " bytes");
    }
    for (int64_t r = 0; r < R; ++r)
        for (int32_t i = 0; i < n; ++i) {
            const void* p = grad_ptrs[r * n + i];
            if (numel[i] > 0 && !p) return fail_without_context(DDP_ERR_ARG, "ddp_sync_static: null gradient pointer");
            if ((reinterpret_cast<uintptr_t>(p) & static_cast<uintptr_t>(ddp::elem_size(dtype[i]) - 1)) != 0)
                return fail_without_context(DDP_ERR_ARG, "ddp_sync_static: gradient pointer not aligned to its element size");
        }
    plan.assign(cap_bytes, nullptr);
    ddp::HostTables ht;
    uintptr_t shift_of[DDP_MAX_REPLICAS];
    int64_t first = 0;
    const uintptr_t* const shift = replicas_alike(plan, grad_ptrs, R, shift_of, &first) ? shift_of : nullptr;
    ddp::build_layout(plan, grad_ptrs, R, ht, nullptr, shift);
    const int32_t nb = static_cast<int32_t>(plan.buckets.size());
    const int64_t ntiles = ht.tile0[n];

    // layout of the scratch array: [segment records | pointer rows | tile map | pad to 256 | R + 1 slabs]
    const size_t seg_bytes = sizeof(ddp::SegInfo) * static_cast<size_t>(n);
    // (eight entries of padding: a row that is read sixteen wide reaches into the tile map and the slabs behind it)
    const size_t ptr_bytes = sizeof(void*) * (static_cast<size_t>(R) * static_cast<size_t>(n) + 8);
    const size_t map_bytes = sizeof(int32_t) * static_cast<size_t>(ntiles);
    const size_t table_bytes = static_cast<size_t>(ddp::round_up_to(static_cast<int64_t>(seg_bytes + ptr_bytes + map_bytes), 256));
    const size_t slab_bytes = static_cast<size_t>(ht.slab_stride) * static_cast<size_t>(R + 1);
    if (table_bytes + slab_bytes > DDP_STATIC_SCRATCH_BYTES)
        return fail_without_context(DDP_ERR_UNSUPPORTED,
                    "ddp_sync_static: tables and flat buckets need " + std::to_string(table_bytes + slab_bytes) +
                    " bytes, the static scratch buffer holds " + std::to_string(DDP_STATIC_SCRATCH_BYTES));

    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK0(hipSetDevice(device));
    const ddp::Scale sc = ddp::make_scale(R);

    // Nobody sees the flat buckets of this call, so the averages go straight into replica 0's
    // tensors: (R + 1) b bytes in one launch per run of buckets of one element type, instead of a
    // fill, the copies, a reduction per bucket and the write-back, (4 R + 5) b in all.  The bits are
    // the same.  A tensor that is written while another block still reads it (one tensor under two
    // parameters or as two replicas) must not be seen half averaged: such lists take the flat buckets.
    // The first 48 ResNet-50 tensors, R = 4: 37 -> 25 us a call; 2e6 elements, R = 2: 50 -> 20.  Many
    // replicas (host arrays ready, flat buckets / so): R = 17, 500 bfloat16 elements in three tensors 18 / 9.0; R = 32,
    // 100000 in thirty 32 / 20; R = 64, 500 22 / 10, 39000 in thirty 46 / 34; binary32, R = 64, 100000 56 / 33.
    const bool in_place = writes_are_apart(plan, grad_ptrs, R, shift);
    auto for_each_run = [&](auto launch_tiles) -> hipError_t {       // in bucket order (Section 3.2.3)
        for (int32_t b = 0; b < nb;) {
            int32_t e = b + 1;
            while (e < nb && plan.buckets[e].dtype == plan.buckets[b].dtype) ++e;
            const int64_t tile0 = ht.tile0[plan.buckets[b].seg_begin];
            const int64_t tile1 = e < nb ? ht.tile0[plan.buckets[e].seg_begin] : ntiles;
            const int64_t nslices = ht.slices[e < nb ? plan.buckets[e].seg_begin : n] - ht.slices[plan.buckets[b].seg_begin];
            const hipError_t err = launch_tiles(plan.buckets[b].dtype, tile0, tile1 - tile0, nslices);
            if (err != hipSuccess) return err;
            b = e;
        }
        return hipSuccess;
    };
    // Tables of up to 448 words travel in the arguments of the kernel that uses them: 2 n + R words where the replicas lie
    // alike, else n (R + 1).  (Written to the scratch array they take a launch for every 3 KiB, each of 3.8 us of the host, and as many
    // hand-overs.)  Us a call, written / by value: R = 2, four tensors 6.1 / 4.5; R = 24, 24 tensors 15.3 / 10.2, 44 25.2 / 14.2; R = 16, 20
    // tensors 12.3 / 7.7; R = 64, 59 tensors 70 / 38 (the list's way through Python is 35 of them); the first 48 ResNet-50 tensors, R = 4,
    // 11.6 / 7.3 (16.1 / 7.3 in another process); 2e6 elements, R = 2 10.8 / 6.7.
    ddp::WordTables by_value{nullptr, n, shift != nullptr};
    if (in_place && by_value.count(R) <= ddp::kTableWords) {
        uint64_t words[ddp::kTableWords];
        by_value.words = words;
        const uintptr_t base0 = reinterpret_cast<uintptr_t>(grad_ptrs[first]);
        for (int32_t g = 0; g < n; ++g) {
            const ddp::SegInfo& si = ht.seg[g];          // (numel < 2^24, the scratch array's limit)
            words[g] = static_cast<uint64_t>(si.numel) | static_cast<uint64_t>(si.congruent() ? 1 : 0) << 31 | static_cast<uint64_t>(si.tile0) << 32;
            if (shift != nullptr) words[n + R + g] = reinterpret_cast<uintptr_t>(grad_ptrs[si.param]) - base0;
            else for (int64_t r = 0; r < R; ++r) words[n + static_cast<int64_t>(g) * R + r] = reinterpret_cast<uintptr_t>(grad_ptrs[r * n + si.param]);
        }
        for (int32_t r = 0; shift != nullptr && r < R; ++r) words[n + r] = base0 + shift[r];
        HIPCHK0(for_each_run([&](int32_t dt, int64_t tile0, int64_t count, int64_t nslices) {
            return ddp::launch_fused_reduce_by_value(dt, by_value, tile0, count, nslices, R, sc, s);
        }));
        return nb;
    }

    unsigned char* base = nullptr;
    HIPCHK0(scratch_on(device, &base));
    ddp::build_host_tables(plan, grad_ptrs, R, ht);
    std::vector<unsigned char> host(seg_bytes + ptr_bytes + map_bytes);
    std::memcpy(host.data(), ht.seg.data(), seg_bytes);
    std::memcpy(host.data() + seg_bytes, ht.grad.data(), ptr_bytes);
    if (map_bytes) std::memcpy(host.data() + seg_bytes + ptr_bytes, ht.tile_seg.data(), map_bytes);
    HIPCHK0(upload(base, host.data(), host.size(), s));

    ddp::SegTables t{};
    t.seg = reinterpret_cast<const ddp::SegInfo*>(base);
    t.grad = reinterpret_cast<void* const*>(base + seg_bytes);
    t.tile_seg = reinterpret_cast<const int32_t*>(base + seg_bytes + ptr_bytes);
    t.G = n;
    t.R = R;
    char* slabs = reinterpret_cast<char*>(base + table_bytes);

    if (in_place) {
        HIPCHK0(for_each_run([&](int32_t dt, int64_t tile0, int64_t count, int64_t nslices) {
            return ddp::launch_fused_reduce(dt, t, tile0, count, 0, nslices, R, 1, ddp::Masks{}, false, sc, true, 0, ddp::FlatBuckets{nullptr, 0}, nullptr, 0,
                                            ddp::DispatchSignal{nullptr, 0}, s);
        }));
        return nb;
    }
    // The array keeps what the previous call left in it.  The flat buckets are
    // rewritten by the pack kernel except for the padding between them, which the
    // reduce kernel reads (whole 16-byte vectors): clear the slabs.
    {
        const int64_t nvec = static_cast<int64_t>(slab_bytes / 16);
        int64_t blocks = (nvec + 255) / 256;
        if (blocks > 2048) blocks = 2048;
        if (blocks > 0) {
            hipLaunchKernelGGL(clear_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                               reinterpret_cast<u32x4*>(slabs), nvec);
            HIPCHK0(hipGetLastError());
        }
    }
    HIPCHK0(ddp::launch_pack(t, 0, ntiles, slabs, ht.slab_stride, R, nullptr, nullptr, 0, s));
    char* out = slabs + static_cast<int64_t>(R) * ht.slab_stride;
    for (int32_t b = 0; b < nb; ++b)      // in bucket order (Section 3.2.3)
        HIPCHK0(ddp::launch_flat_reduce(plan.buckets[b].dtype, slabs + ht.bucket_slab_off[b], ht.slab_stride,
                                        out + ht.bucket_slab_off[b], ht.bucket_vecs[b], R, sc, true, 0, nullptr, 0,
                                        ddp::DispatchSignal{nullptr, 0}, s));
    HIPCHK0(ddp::launch_unpack(t, 0, ntiles, out, 1, nullptr, false, s));
    return nb;
}
