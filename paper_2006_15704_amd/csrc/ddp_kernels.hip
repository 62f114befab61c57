// HIP kernels of the bucketed gradient synchronization path, written for
// gfx950 (MI355X): 64-wide wavefronts, 16-byte vector loads, fp32
// accumulation in registers.  The path is a streaming reduction (about one
// add per four bytes read), so every kernel here is bound by HBM bandwidth
// and none uses the matrix cores.
//
// Paper anchors: pack = the copy of a gradient into its bucket view
// (Algorithm 1, autograd_hook); reduce = the bucket AllReduce (Section 2.3:
// sum over participants) followed by DDP's averaging (Section 3.2.1); unpack
// = the finalizing write-back described after Algorithm 1; accumulate = the
// local gradient accumulation of no_sync (Section 3.2.4).
#include "ddp_kernels.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <set>
#include <type_traits>
#include <utility>

namespace ddp {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Every gradient, slab and table lives in global memory.  Pointers that are
// read from tables carry no address space, and the compiler would fall back to
// generic (flat) accesses for them; the casts below keep all traffic on the
// global path.
#define DDP_GLOBAL __attribute__((address_space(1)))
typedef DDP_GLOBAL const u32x4* gc_u32x4;
typedef DDP_GLOBAL u32x4* g_u32x4;

template <typename T>
__device__ __forceinline__ T gload(const char* p) {
    return *(DDP_GLOBAL const T*)(p);
}
template <typename T>
__device__ __forceinline__ void gstore(char* p, T v) {
    *(DDP_GLOBAL T*)(p) = v;
}

template <bool NT>
__device__ __forceinline__ u32x4 load16(const char* p) {
    gc_u32x4 q = (gc_u32x4)(p);
    if (NT) return __builtin_nontemporal_load(q);
    return *q;
}
__device__ __forceinline__ void store16(char* p, u32x4 v) {
    *(g_u32x4)(p) = v;
}
// Results that are not read again soon are stored with the non-temporal hint.
template <bool NT>
__device__ __forceinline__ void store16s(char* p, u32x4 v) {
    if (NT) __builtin_nontemporal_store(v, (g_u32x4)(p));
    else *(g_u32x4)(p) = v;
}
__device__ __forceinline__ u32x4 zero16() {
    u32x4 z = {0u, 0u, 0u, 0u};
    return z;
}
// 16 bytes at an address that is only element-aligned (2 or 4 bytes): gfx950
// serves such an access with one vector instruction too, so a tensor that sits
// off the 16-byte grid of its peers costs extra cache lines, not a scalar loop.
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef uint32_t u32_a2 __attribute__((aligned(2)));
template <bool NT>
__device__ __forceinline__ u32x4 load16u(const char* p) {
    DDP_GLOBAL const u32x4_a2* q = (DDP_GLOBAL const u32x4_a2*)(p);
    if (NT) return __builtin_nontemporal_load(q);
    return *q;
}
template <bool NT>
__device__ __forceinline__ void store16u(char* p, u32x4 v) {
    DDP_GLOBAL u32x4_a2* q = (DDP_GLOBAL u32x4_a2*)(p);
    if (NT) __builtin_nontemporal_store(v, q);
    else *q = v;
}

// Tables, masks and gate records do not change while a kernel runs that reads them here, and a block reads
// them at uniform addresses: through the constant address space these are scalar loads, which the compiler may
// also move and merge.  (As plain loads it kept them behind the atomic of signal_dispatch, as vector loads with
// a v_readfirstlane for every word, and waited for some before it issued the next.)
// The kernel alone, us, two tensors, plain / scalar: binary32, 512 tiles R = 8 9.5 / 8.4, R = 16 16.2 / 14.0, R = 32
// 28.6 / 26.0, R = 64 55 / 49; slices, 256 tiles R = 32 17.3 / 12.5, R = 64 32 / 23; bfloat16, 256 tiles R = 16 10.1 / 9.0.
// The ragged list, R = 8, 199 / 197 us.  Whole tiles in long launches are another matter, see fused_tile.
#define DDP_CONSTANT __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ T cload(const T* p) {
    return *(DDP_CONSTANT const T*)(p);
}
__device__ __forceinline__ SegInfo segment(const SegTables& t, int g) {
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
    static_assert(sizeof(SegInfo) == sizeof(u32x8), "one scalar load");
    return __builtin_bit_cast(SegInfo, *(DDP_CONSTANT const u32x8*)(t.seg + g));
}
struct PointerRow {                        // a segment's R pointers
    DDP_CONSTANT const uint64_t* p;
    __device__ __forceinline__ char* operator[](int r) const { return reinterpret_cast<char*>(p[r]); }
};
__device__ __forceinline__ PointerRow pointer_row(void* const* table, int g, int R) {
    return PointerRow{(DDP_CONSTANT const uint64_t*)(table + static_cast<int64_t>(g) * R)};
}
__device__ __forceinline__ int segment_of(const SegTables& t, int64_t tile) { return cload(t.tile_seg + tile); }
__device__ __forceinline__ PointerRow gradients_of(const SegTables& t, int g) { return pointer_row(t.grad, g, t.R); }

// Which slice a block of a slice launch takes, as tile * SLICES + slice (base: of the launch's tiles, or of its listed slices).
__device__ __forceinline__ int64_t slice_of(const SegTables& t, int64_t base, int block) {
    return t.slices != nullptr ? cload(t.slices + base + block) : base * SLICES + block;
}

// Tables that travel in the launch's arguments (WordTables has the layout).  There is no tile map: a wave compares the first
// tiles of 64 segments with its own at a time.
template <int N>
struct ArgTables {
    uint64_t w[N + 16];                    // (a row is read up to sixteen entries wide)
    int32_t n, R;
    int32_t at, step;                      // the pointers of segment g start at w[at + g * step] ...
    int32_t dist;                          // ... and, if this is not 0, lie w[dist + g] further on
};
template <int N>
struct ArgRow {
    const ArgTables<N>& t;
    int at;
    uint64_t dist;
    __device__ __forceinline__ char* operator[](int r) const { return reinterpret_cast<char*>(t.w[at + r] + dist); }
};
template <int N>
__device__ __forceinline__ int segment_of(const ArgTables<N>& t, int64_t tile) {
    const int lane = threadIdx.x & 63;
    int before = 0;
    for (int g = 0; g < t.n; g += 64) {
        const int i = min(g + lane, t.n - 1);
        const bool starts = g + lane < t.n && static_cast<int64_t>(t.w[i] >> 32) <= tile;
        before += __popcll(__ballot(starts));
    }
    return __builtin_amdgcn_readfirstlane(before - 1);     // (segments without elements share the next one's first tile)
}
template <int N>
__device__ __forceinline__ int64_t slice_of(const ArgTables<N>&, int64_t base, int block) { return base * SLICES + block; }
template <int N>
__device__ __forceinline__ ArgRow<N> gradients_of(const ArgTables<N>& t, int g) {
    return ArgRow<N>{t, t.at + g * t.step, t.dist != 0 ? t.w[t.dist + g] : 0};
}
template <int N>
__device__ __forceinline__ SegInfo segment(const ArgTables<N>& t, int g) {
    const uint64_t w = t.w[g];
    SegInfo si;
    si.numel = static_cast<uint32_t>(w) & 0x7FFFFFFFu;
    si.tile0 = static_cast<int64_t>(w >> 32);
    si.flat_byte = 0;
    si.param = 0;
    si.flags = (static_cast<uint32_t>(w) >> 31 ? 0x100 : 0) | static_cast<int>(reinterpret_cast<uintptr_t>(gradients_of(t, g)[0]) & 15u) << 16;
    return si;
}

// Where a launch's participation masks are (Masks).  In the arguments they spare it the kernel that writes them to the table:
// one launch of three or four less for the host (3.8 us), and a hand-over on the stream (2.5 us) in front of the reduction.
// One mark per call, us a synchronization, table / arguments: ResNet-50, R = 8, 0.7 of the flags set 140 / 134; 300000 elements in forty 32 KiB
// buckets, R = 8 348 / 165 to 210; bfloat16, 6 MB in seven buckets, R = 4 85 / 47 to 60; 2 MiB buckets, R = 8 82 / 58 to 68; a tenth of the parameters
// never marked, R = 4, 0.4 MB 18.9 / 14.2; all marks in one call, binary16, R = 8, 20 MB 36.6 / 33.1.
struct NoMasks {
    static constexpr bool ANY = false;
    __device__ __forceinline__ bool present() const { return false; }
    __device__ __forceinline__ uint64_t of(int) const { return 0; }
};
struct MaskTable {
    static constexpr bool ANY = true;
    const uint64_t* local;                 // null: every replica used every parameter
    __device__ __forceinline__ bool present() const { return local != nullptr; }
    __device__ __forceinline__ uint64_t of(int g) const { return cload(local + g); }
};
struct MaskWords {
    static constexpr bool ANY = true;
    uint64_t m[kMaskWords];
    int32_t first, shift;
    __device__ __forceinline__ bool present() const { return true; }
    __device__ __forceinline__ uint64_t of(int g) const {
        const int bit = (g - first) << shift;
        const uint64_t w = m[bit >> 6];
        return shift == 6 ? w : (w >> (bit & 63)) & ((uint64_t(1) << (1 << shift)) - 1);
    }
};

// ---- element formats ------------------------------------------------------
template <int DT> struct Fmt;

template <> struct Fmt<0> {   // binary32
    static constexpr int ES = 4, VEC = 4;
    static __device__ __forceinline__ void widen(u32x4 v, float (&f)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(v[i]);
    }
    static __device__ __forceinline__ u32x4 narrow(const float (&f)[4]) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(f[i]);
        return v;
    }
    static __device__ __forceinline__ float value(uint32_t bits) { return __uint_as_float(bits); }
    static __device__ __forceinline__ float load1(const char* p) {
        return gload<float>(p);
    }
    static __device__ __forceinline__ void store1(char* p, float y) {
        gstore<float>(p, y);
    }
};

template <> struct Fmt<1> {   // binary16: exact widening, round-to-nearest-even narrowing
    static constexpr int ES = 2, VEC = 8;
    static __device__ __forceinline__ float up(uint32_t bits16) {
        return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(bits16)));
    }
    static __device__ __forceinline__ uint32_t down(float y) {
        return __builtin_bit_cast(uint16_t, static_cast<_Float16>(y));
    }
    static __device__ __forceinline__ void widen(u32x4 v, float (&f)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = up(v[i] & 0xFFFFu);
            f[2 * i + 1] = up(v[i] >> 16);
        }
    }
    static __device__ __forceinline__ u32x4 narrow(const float (&f)[8]) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = down(f[2 * i]) | (down(f[2 * i + 1]) << 16);
        return v;
    }
    static __device__ __forceinline__ float value(uint32_t bits) { return up(bits); }
    static __device__ __forceinline__ float load1(const char* p) {
        return up(gload<uint16_t>(p));
    }
    static __device__ __forceinline__ void store1(char* p, float y) {
        gstore<uint16_t>(p, static_cast<uint16_t>(down(y)));
    }
};

template <> struct Fmt<2> {   // bfloat16 = upper half of binary32
    static constexpr int ES = 2, VEC = 8;
    static __device__ __forceinline__ uint32_t down(float y) {
        uint32_t u = __float_as_uint(y);
        if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x0040u;   // NaN stays NaN
        u += 0x7FFFu + ((u >> 16) & 1u);                                     // nearest, ties to even
        return u >> 16;
    }
    static __device__ __forceinline__ void widen(u32x4 v, float (&f)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(v[i] << 16);
            f[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
        }
    }
    static __device__ __forceinline__ u32x4 narrow(const float (&f)[8]) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = down(f[2 * i]) | (down(f[2 * i + 1]) << 16);
        return v;
    }
    static __device__ __forceinline__ float value(uint32_t bits) { return __uint_as_float(bits << 16); }
    static __device__ __forceinline__ float load1(const char* p) {
        return value(gload<uint16_t>(p));
    }
    static __device__ __forceinline__ void store1(char* p, float y) {
        gstore<uint16_t>(p, static_cast<uint16_t>(down(y)));
    }
};

__device__ __forceinline__ float apply_scale(const Scale& sc, float s) {
    return sc.use_mul ? s * sc.mul : s / sc.div;
}

// Vectors are cut at 16-byte boundaries of the destination.  `sh` elements
// precede the segment start inside the first vector, so element index
// e = tile_elem - sh may be negative for the first vector of a segment.
__device__ __forceinline__ int lead_in(const void* dst, int es) {
    return static_cast<int>(reinterpret_cast<uintptr_t>(dst) & 15u) / es;
}
__device__ __forceinline__ bool congruent16(const void* a, const void* b) {
    return ((reinterpret_cast<uintptr_t>(a) ^ reinterpret_cast<uintptr_t>(b)) & 15u) == 0;
}

enum { V_NONE = 0, V_FULL = 1, V_EDGE = 2 };
__device__ __forceinline__ int classify(int64_t e, int vec, int64_t numel) {
    if (e >= numel) return V_NONE;
    return (e >= 0 && e + vec <= numel) ? V_FULL : V_EDGE;
}

// The last block of the grid tells that the launch has been dispatched in full (blocks start
// in index order): a launch chained behind this one may begin to fill the compute units
// (reporting a few hundred blocks earlier, to make up for the start-up of the next launch,
// measured no better; 1024 and more blocks earlier lose the gain).
__device__ __forceinline__ void signal_dispatch(const DispatchSignal& sig) {
    if (sig.word != nullptr && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        __hip_atomic_fetch_max(sig.word, sig.ord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- K1 / K3: segment copies ---------------------------------------------
template <int ES>
__device__ __forceinline__ void copy_tile(const char* __restrict__ src, char* __restrict__ dst,
                                          int64_t numel, int64_t ltile, bool zero) {
    constexpr int VEC = 16 / ES;
    constexpr int U = TILE_VECS / BLOCK;
    const int sh = lead_in(dst, ES);
    const bool cong = congruent16(src, dst);
    const int64_t e_tile = ltile * (TILE_BYTES / ES) - sh;
    int64_t e[U];
    int kind[U];
    u32x4 v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        e[k] = e_tile + static_cast<int64_t>(k * BLOCK + threadIdx.x) * VEC;
        kind[k] = classify(e[k], VEC, numel);
        v[k] = zero16();
        if (kind[k] == V_FULL && !zero)
            v[k] = cong ? load16<true>(src + e[k] * ES) : load16u<true>(src + e[k] * ES);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
        if (kind[k] == V_FULL) {
            store16(dst + e[k] * ES, v[k]);
        } else if (kind[k] == V_EDGE) {
            for (int i = 0; i < VEC; ++i) {
                const int64_t idx = e[k] + i;
                if (idx < 0 || idx >= numel) continue;
                if (ES == 4) {
                    gstore<uint32_t>(dst + idx * 4, zero ? 0u : gload<uint32_t>(src + idx * 4));
                } else {
                    gstore<uint16_t>(dst + idx * 2, zero ? uint16_t(0) : gload<uint16_t>(src + idx * 2));
                }
            }
        }
    }
}

// PACK: grad[r][g] -> slab_r + flat_byte[g];  UNPACK: out slab -> grad[r][g].
// GATED: the launch has a gate in front of it (PACK only; see fused_tile).
template <bool PACK, bool GATED>
__global__ __launch_bounds__(BLOCK) void seg_copy_kernel(SegTables t, int64_t tile_base,
                                                         char* slab0, int64_t slab_stride,
                                                         const uint64_t* __restrict__ local,
                                                         const uint8_t* __restrict__ global_used,
                                                         int keep_unused,
                                                         const GateRecord* __restrict__ gate, uint32_t tag) {
    if (GATED && cload(&gate->failed_tag) == tag) return;
    const int64_t tile = tile_base + blockIdx.x;
    const int r = blockIdx.y;
    const int g = cload(t.tile_seg + tile);
    const SegInfo si = segment(t, g);
    const int64_t numel = si.numel;
    const int64_t ltile = tile - si.tile0;
    char* grad = pointer_row(t.grad, g, t.R)[r];
    // PACK: local = participation masks, bit r = 0: the replica did not use the
    // parameter, its slot gets zeros and its tensor is not read.
    // UNPACK: global_used[g] = 0: no replica used the parameter, with keep_unused
    // its gradients are left as they are.
    const bool zero = PACK && local != nullptr && ((cload(local + g) >> r) & 1u) == 0;
    if (!PACK && keep_unused && global_used != nullptr && cload(global_used + g) == 0) return;
    const char* src;
    char* dst;
    if (PACK) {
        src = grad;
        dst = slab0 + r * slab_stride + si.flat_byte;
    } else {
        src = slab0 + si.flat_byte;
        dst = grad;
    }
    if (si.dtype() == 0) copy_tile<4>(src, dst, numel, ltile, zero);
    else copy_tile<2>(src, dst, numel, ltile, zero);
}

// ---- K2: reduce and average ------------------------------------------------
// acc += widen(x), elementwise, in the order the calls are made.
template <int DT>
__device__ __forceinline__ void add_into(float (&acc)[Fmt<DT>::VEC], u32x4 x) {
    float f[Fmt<DT>::VEC];
    Fmt<DT>::widen(x, f);
#pragma unroll
    for (int i = 0; i < Fmt<DT>::VEC; ++i) acc[i] += f[i];
}

// Interior work (every vector of the block lies inside the data): no lane is
// predicated.  base_of(r) returns replica r's block-uniform base address, which
// need only be element-aligned; the per-thread part of the address is a 32-bit
// byte offset, so the loads take the scalar-base + vector-offset form.  All C*U
// loads are issued before the adds, which run in ascending r.  (The instruction
// is the same for any alignment; a base off the 16-byte grid costs one more
// cache line per wave and load, which the non-temporal hint does not evict
// before the neighbouring wave has used it: plain loads were 7 % slower.)
template <int DT, bool NT, int C, int U, typename BaseFn>
__device__ __forceinline__ void chunk_interior(BaseFn base_of, int r, const uint32_t (&lane_off)[U],
                                               float (&acc)[U][Fmt<DT>::VEC]) {
    const char* base[C];
#pragma unroll
    for (int i = 0; i < C; ++i) base[i] = base_of(r + i);
    u32x4 x[C][U];
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u) x[i][u] = load16u<NT>(base[i] + lane_off[u]);
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u) add_into<DT>(acc[u], x[i][u]);
}

// The same for a tile that is also copied into the replicas' flat buckets (staged pipeline): slot is
// the tile's place in replica r's buffer, `used` says whose tensors are read; a replica that did not
// use the parameter contributes zeros to its bucket and to the sum.
// Bound by HBM: a bucket of b bytes costs R b read and (R + 1) b written in this one pass, where packing
// and reducing in two kernels read the copies back ((2 R + 1) b instead of (3 R + 1) b in all).
// ResNet-50, R = 8, one call for all marks: 477 -> 375 us a synchronization including the write-back;
// the copies are not read again on the path, and without the non-temporal hint on them it is 402 us.
template <int DT, bool NT, int C, int U>
__device__ __forceinline__ void chunk_copy(void* const* __restrict__ row, int r, uint64_t used, int64_t tile_byte,
                                           char* slot, int64_t stride, const uint32_t (&lane_off)[U],
                                           float (&acc)[U][Fmt<DT>::VEC]) {
    const char* base[C];
#pragma unroll
    for (int i = 0; i < C; ++i) base[i] = static_cast<const char*>(row[r + i]) + tile_byte;
    u32x4 x[C][U];
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const bool take = ((used >> (r + i)) & 1u) != 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[i][u] = zero16();
            if (take) x[i][u] = load16u<NT>(base[i] + lane_off[u]);
        }
    }
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            store16s<NT>(slot + i * stride + lane_off[u], x[i][u]);
            add_into<DT>(acc[u], x[i][u]);
        }
}

// The last `left` (0..7) replicas as ONE chunk, so that all of their loads are
// in flight together (a 4 + 2 + 1 split would run three dependent phases).
template <int DT, bool NT, int U, typename BaseFn>
__device__ __forceinline__ void tail_interior(BaseFn base_of, int r, int left,
                                              const uint32_t (&lane_off)[U],
                                              float (&acc)[U][Fmt<DT>::VEC]) {
    switch (left) {
        case 7: chunk_interior<DT, NT, 7, U>(base_of, r, lane_off, acc); break;
        case 6: chunk_interior<DT, NT, 6, U>(base_of, r, lane_off, acc); break;
        case 5: chunk_interior<DT, NT, 5, U>(base_of, r, lane_off, acc); break;
        case 4: chunk_interior<DT, NT, 4, U>(base_of, r, lane_off, acc); break;
        case 3: chunk_interior<DT, NT, 3, U>(base_of, r, lane_off, acc); break;
        case 2: chunk_interior<DT, NT, 2, U>(base_of, r, lane_off, acc); break;
        case 1: chunk_interior<DT, NT, 1, U>(base_of, r, lane_off, acc); break;
        default: break;
    }
}

template <int DT, bool NT, int U, typename BaseFn>
__device__ __forceinline__ void sum_interior(BaseFn base_of, int R, const uint32_t (&lane_off)[U],
                                             float (&acc)[U][Fmt<DT>::VEC]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < Fmt<DT>::VEC; ++i) acc[u][i] = -0.0f;   // -0 + x == x for every x
    int r = 0;
    for (; r + 8 <= R; r += 8) chunk_interior<DT, NT, 8, U>(base_of, r, lane_off, acc);
    tail_interior<DT, NT, U>(base_of, r, R - r, lane_off, acc);
}

// The same with the first eight replica pointers already in registers (they are
// fetched together with the segment record, one dependent memory access
// earlier than a fetch inside the loop would be).
template <int DT, bool NT, int U, typename BaseFn>
__device__ __forceinline__ void sum_interior_pre(const char* const (&pre)[8], int64_t byte0,
                                                 BaseFn base_of, int R,
                                                 const uint32_t (&lane_off)[U],
                                                 float (&acc)[U][Fmt<DT>::VEC]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < Fmt<DT>::VEC; ++i) acc[u][i] = -0.0f;
    int r = 0;
    if (R >= 8) {
        chunk_interior<DT, NT, 8, U>([&](int k) { return pre[k] + byte0; }, 0, lane_off, acc);
        r = 8;
    }
    for (; r + 8 <= R; r += 8) chunk_interior<DT, NT, 8, U>(base_of, r, lane_off, acc);
    if (r == 0) {
        // fewer than eight replicas: their pointers are the preloaded ones
        tail_interior<DT, NT, U>([&](int k) { return pre[k] + byte0; }, 0, R, lane_off, acc);
    } else {
        tail_interior<DT, NT, U>(base_of, r, R - r, lane_off, acc);
    }
}

// A tile of a parameter that only some replicas used: their tensors alone are read, in ascending
// order.  Each of the others counts as +0, and there is at least one: a running sum that starts at
// +0 differs from the sum with those +0 in their places only in the sign of a zero in between, and
// both end in +0 where the sum is zero.
template <int DT, bool NT, int U>
__device__ __forceinline__ void sum_interior_used(PointerRow row, int64_t byte0, uint64_t used,
                                                  const uint32_t (&lane_off)[U],
                                                  float (&acc)[U][Fmt<DT>::VEC]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < Fmt<DT>::VEC; ++i) acc[u][i] = 0.0f;
    uint64_t rest = used;
    auto next = [&](int) {
        const int r = __builtin_ctzll(rest);
        rest &= rest - 1;
        return row[r] + byte0;
    };
    int left = __popcll(used);
    for (; left >= 8; left -= 8) chunk_interior<DT, NT, 8, U>(next, 0, lane_off, acc);
    tail_interior<DT, NT, U>(next, 0, left, lane_off, acc);
}

template <int DT>
__device__ __forceinline__ u32x4 scaled(const Scale& sc, const float (&acc)[Fmt<DT>::VEC]) {
    float y[Fmt<DT>::VEC];
#pragma unroll
    for (int i = 0; i < Fmt<DT>::VEC; ++i) y[i] = apply_scale(sc, acc[i]);
    return Fmt<DT>::narrow(y);
}

// C replicas starting at r, U vectors per thread: issue all C*U loads, then
// add them in ascending r.
template <int DT, bool NT, int C, int U>
__device__ __forceinline__ void chunk_flat(const char* __restrict__ in0, int64_t stride, int r,
                                           const int64_t (&off)[U], const bool (&ok)[U],
                                           float (&acc)[U][Fmt<DT>::VEC]) {
    u32x4 x[C][U];
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const char* p = in0 + static_cast<int64_t>(r + i) * stride;
#pragma unroll
        for (int u = 0; u < U; ++u) x[i][u] = ok[u] ? load16<NT>(p + off[u]) : zero16();
    }
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u) add_into<DT>(acc[u], x[i][u]);
}

// Every block handles one row of BLOCK*U consecutive vectors, so blocks stream
// through memory in launch order (a bounded grid whose blocks loop over distant
// rows measured slower).
// GATED: gate or sig are set (without them the kernel starts without a look at either).
template <int DT, bool NT, int U, bool GATED>
__global__ __launch_bounds__(BLOCK) void flat_reduce_kernel(const char* __restrict__ in0,
                                                            int64_t stride, char* __restrict__ out,
                                                            int64_t nvec, int R, Scale sc,
                                                            const GateRecord* __restrict__ gate,
                                                            uint32_t tag, DispatchSignal sig) {
    constexpr int VEC = Fmt<DT>::VEC;
    if (GATED) {
        signal_dispatch(sig);
        if (gate != nullptr && cload(&gate->failed_tag) == tag) return;
    }
    const int64_t row = blockIdx.x;
    float acc[U][VEC];
    if ((row + 1) * (BLOCK * U) <= nvec) {
        const int64_t row_byte = row * (BLOCK * U * 16);
        uint32_t lane_off[U];
#pragma unroll
        for (int u = 0; u < U; ++u) lane_off[u] = (u * BLOCK + threadIdx.x) * 16u;
        sum_interior<DT, NT, U>(
            [&](int r) { return in0 + static_cast<int64_t>(r) * stride + row_byte; }, R, lane_off, acc);
#pragma unroll
        for (int u = 0; u < U; ++u)
            store16s<NT>(out + row_byte + lane_off[u], scaled<DT>(sc, acc[u]));
        return;
    }
    int64_t off[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t v = row * (BLOCK * U) + u * BLOCK + threadIdx.x;
        ok[u] = v < nvec;
        off[u] = v * 16;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[u][i] = -0.0f;   // -0 + x == x for every x
    }
    int r = 0;
    for (; r + 8 <= R; r += 8) chunk_flat<DT, NT, 8, U>(in0, stride, r, off, ok, acc);
    if (r + 4 <= R) { chunk_flat<DT, NT, 4, U>(in0, stride, r, off, ok, acc); r += 4; }
    if (r + 2 <= R) { chunk_flat<DT, NT, 2, U>(in0, stride, r, off, ok, acc); r += 2; }
    if (r < R) { chunk_flat<DT, NT, 1, U>(in0, stride, r, off, ok, acc); }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!ok[u]) continue;
        float y[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) y[i] = apply_scale(sc, acc[u][i]);
        store16s<NT>(out + off[u], Fmt<DT>::narrow(y));
    }
}

// Fused variant, boundary tiles: replica pointers come from the segment table
// and lanes are predicated.  The C pointers are fetched first (one scalar
// load), then all C*U vector loads are issued, then the adds run in order.
// With `slot` set (staged pipeline) the vectors also go to the replicas' flat buckets.
template <int DT, bool NT, int C, int U, typename Row>
__device__ __forceinline__ void chunk_seg(const Row& row, int r, uint64_t used, bool aligned,
                                          const int64_t (&off)[U], const bool (&ok)[U],
                                          float (&acc)[U][Fmt<DT>::VEC], char* slot = nullptr, int64_t stride = 0) {
    const char* base[C];
#pragma unroll
    for (int i = 0; i < C; ++i) base[i] = row[r + i];
    u32x4 x[C][U];
    // a replica that did not use the parameter contributes +0 in its place in
    // the sum, and its tensor is not read
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u)
            x[i][u] = (ok[u] && ((used >> (r + i)) & 1u))
                          ? (aligned ? load16<NT>(base[i] + off[u]) : load16u<NT>(base[i] + off[u]))
                          : zero16();
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (slot != nullptr && ok[u]) store16s<NT>(slot + (r + i) * stride + off[u], x[i][u]);
            add_into<DT>(acc[u], x[i][u]);
        }
}

// Where the averages go.  OUT_GRAD: into the gradient tensors themselves, in their
// own format (replica 0's, or all of them).  OUT_BINARY32: the gradients are a
// 16-bit transport format (Section 6.2.3) and the averages are written as
// binary32, unrounded, to a separate tensor per parameter (SegTables::out): two
// 16-byte stores per 16-byte input vector, at twice the byte offset.  OUT_FLAT
// (staged pipeline): every replica's gradients are copied into its flat bucket
// buffer and the average goes to the averaged bucket (FlatBuckets).
enum { OUT_GRAD = 0, OUT_BINARY32 = 1, OUT_FLAT = 2 };

template <int DT, bool NT>
__device__ __forceinline__ void store_out32(char* out, int64_t in_byte_off, const float (&y)[Fmt<DT>::VEC],
                                            bool aligned = true) {
    static_assert(Fmt<DT>::VEC == 8, "binary32 outputs are for the 16-bit formats");
    u32x4 lo, hi;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        lo[i] = __float_as_uint(y[i]);
        hi[i] = __float_as_uint(y[4 + i]);
    }
    if (aligned) {
        store16s<NT>(out + 2 * in_byte_off, lo);
        store16s<NT>(out + 2 * in_byte_off + 16, hi);
    } else {
        store16u<NT>(out + 2 * in_byte_off, lo);
        store16u<NT>(out + 2 * in_byte_off + 16, hi);
    }
}

// The same for a whole wave whose 64 lanes hold 64 consecutive input vectors (interior tiles):
// lane i's eight values belong at bytes [32 i, 32 i + 32) of the wave's 2 KiB of output, which
// two stores per lane at a stride of 32 bytes would write as half cache lines (counters: 10 %
// more bytes written than the averages hold).  The values are exchanged between the lanes
// instead, so that each of the two store instructions writes 1 KiB without gaps: lane i stores
// floats 4 i .. 4 i + 3 of the first KiB, then of the second.
template <int DT, bool NT>
__device__ __forceinline__ void store_out32_wave(char* out, int64_t in_byte_off, const float (&y)[Fmt<DT>::VEC]) {
    static_assert(Fmt<DT>::VEC == 8, "binary32 outputs are for the 16-bit formats");
    const int lane = threadIdx.x & 63;
    char* wave_base = out + 2 * in_byte_off - 32 * lane;
    const int src = lane >> 1;                // the lane whose vector holds floats 4 i .. 4 i + 3
    const bool upper = (lane & 1) != 0;       // ... in its upper half
    u32x4 a, b;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int lo = __float_as_int(y[k]), hi = __float_as_int(y[4 + k]);
        const int a_lo = __shfl(lo, src), a_hi = __shfl(hi, src);
        const int b_lo = __shfl(lo, 32 + src), b_hi = __shfl(hi, 32 + src);
        a[k] = static_cast<uint32_t>(upper ? a_hi : a_lo);
        b[k] = static_cast<uint32_t>(upper ? b_hi : b_lo);
    }
    store16u<NT>(wave_base + 16 * lane, a);
    store16u<NT>(wave_base + 1024 + 16 * lane, b);
}

// The elements of a block's part [e0, e0 + span) of a segment that lie in vectors reaching over an end of
// the segment: the first `head` elements of the segment and the `tail` elements from `last` on, at most
// VEC - 1 each.
struct EdgeElements {
    int head, tail;
    int64_t last;
};
template <int VEC>
__device__ __forceinline__ EdgeElements edge_elements(int64_t e0, int span, int64_t numel) {
    const int64_t rest = numel - e0;                       // elements from the part's start on, at least 1
    EdgeElements ed;
    ed.last = e0 + rest / VEC * VEC;                       // first element of the vector with the segment's end
    ed.head = e0 < 0 ? static_cast<int>(rest < VEC ? numel : VEC + e0) : 0;
    ed.tail = rest < span && ed.last >= 0 ? static_cast<int>(numel - ed.last) : 0;
    return ed;
}

// One tile of the fused gather-reduce-scatter.
// gate / tag: see GateRecord (null = no gate).  A launch whose gate gave up must
// not touch gradients that may still be incomplete; the repair launch redoes it.
// The gate word is fetched together with the tile's tables (one round of scalar
// loads, not one more in front of them) and looked at before any gradient is.
// Masks: most launches have none (NoMasks), and the chunks of 1 to 8
// replicas that sum_interior_used adds make the code a third longer, at the same
// registers: the first 101 BERT-large tensors with masks compiled in / left out, binary16,
// R = 16, one mark per call 681 / 677 us a synchronization; bfloat16, R = 8, 329 / 327, and with
// the averages to every replica 627.5 / 626.5.
// FORM: see table_form.
template <int DT, bool NT, int U, int OUT, typename Masks, int FORM = 0, typename Tables = SegTables>
__device__ __forceinline__ void fused_tile(const Tables& t, int64_t tile, int R, int nwrite,
                                           const Masks& masks, int keep_unused,
                                           const Scale& sc, const FlatBuckets& flat,
                                           const GateRecord* __restrict__ gate = nullptr, uint32_t tag = 0) {
    constexpr int ES = Fmt<DT>::ES;
    constexpr int VEC = Fmt<DT>::VEC;
    constexpr int SPAN = BLOCK * U * VEC;           // elements of a tile
    static_assert(BLOCK * U == TILE_VECS, "a block takes a tile");
    typedef typename std::conditional<ES == 4, uint32_t, uint16_t>::type bits;
    extern __shared__ __align__(16) uint32_t shared_words[];
    bits* const edge = reinterpret_cast<bits*>(shared_words);      // [R][EDGE_SLOTS]
    const uint32_t gate_word = gate != nullptr ? cload(&gate->failed_tag) : ~tag;
    // Everything that depends on g alone is fetched together: the segment
    // record and the first eight replica pointers (the pointer table is padded
    // so that eight entries can always be read).
    // Which of the three accesses are scalar loads decides when a block's first gradient loads go out, and long
    // launches of whole tiles are sensitive to that (a block that starts sooner is not always better: the
    // memory system is full, and how the blocks' requests interleave in it changes).  The first 101 BERT-large tensors, us, all
    // plain / tile map plain, others scalar / all scalar, the best cap on resident blocks each: binary32 R = 3 264 / - / -,
    // R = 4 338 / 352 / 350, R = 8 617 / 617 / 631, R = 16 (60 tensors) 852 / 866 / 864; bfloat16 R = 2 112 / 102 / 98, R = 3 146 / 132 / 134, R = 4
    // 165 / 167 / 176, R = 8 319 / 314 / 306, R = 12 451 / 450 / 453, R = 16 590 / 594 / 597; binary32 averages of BERT-large 1144 / 1138 /
    // 1126 (further forms for long launches: table_form); staged (pointers plain in every case: chunk_copy) binary32 R = 4 540 / - / 529, R = 2 332 / - / 336, bfloat16 R = 2 170 / - / 174.
    constexpr bool IN_MEMORY = std::is_same<Tables, SegTables>::value;
    constexpr bool PLAIN = IN_MEMORY && (ES == 4 || FORM == 2 || (OUT == OUT_BINARY32 && FORM == 1));
    int g;
    if constexpr (IN_MEMORY) g = OUT == OUT_BINARY32 && !PLAIN ? cload(t.tile_seg + tile) : t.tile_seg[tile];
    else g = segment_of(t, tile);
    const auto row = gradients_of(t, g);
    SegInfo si;
    if constexpr (PLAIN) si = t.seg[g];
    else si = segment(t, g);
    const char* pre[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if constexpr (PLAIN) pre[i] = static_cast<const char*>(t.grad[static_cast<int64_t>(g) * t.R + i]);
        else pre[i] = row[i];
    }
    // (behind a gate that gave up this row of a table may be an earlier iteration's: it is not looked at then)
    constexpr bool MASKED = Masks::ANY;
    const bool masked = masks.present();
    const uint64_t mask = masked ? masks.of(g) : 0;
    if (gate_word == tag) return;          // the gate in front of this launch gave up
    const int64_t numel = si.numel;
    // participation of the R replicas in this parameter (bit r = replica r used
    // it); without a flag table every replica did
    const uint64_t everyone = R >= 64 ? ~uint64_t(0) : ((uint64_t(1) << R) - 1);
    const uint64_t used = masked ? mask : everyone;
    if (OUT != OUT_FLAT && used == 0 && keep_unused) return;   // globally unused: the gradients stay as they are
    const bool zero = OUT != OUT_FLAT && used == 0;            // ... or become zeros (flat buckets always do)
    const bool all_used = !MASKED || used == everyone;
    // replica 0's tensor -- or the slot in the flat bucket -- starts this many elements past a 16-byte boundary
    const int sh = (OUT == OUT_FLAT ? static_cast<int>(si.flat_byte & 15) : si.lead_bytes()) / ES;
    const bool src_aligned = si.congruent();   // every replica's tensor sits at the same offset modulo 16
    char* outp = nullptr;
    if constexpr (OUT == OUT_BINARY32) outp = pointer_row(t.out, g, 1)[0];
    char* const slot = OUT == OUT_FLAT ? flat.slab0 + si.flat_byte : nullptr;
    const int64_t e0 = (tile - si.tile0) * SPAN - sh;

    // The whole tile is inside the segment.  Where the replicas sit
    // modulo 16 does not matter: vectors are cut on replica 0's 16-byte grid, the other replicas (and
    // a binary32 output tensor that is off the grid) are accessed with element-aligned vectors.  90
    // densely packed tensors of odd sizes, R = 8, 120 MB each, replicas 4 bytes apart modulo 16: 235 us
    // when such tiles took the predicated path below, 203 us here (5.3 TB/s; 5.9 when congruent).
    if (e0 >= 0 && e0 + SPAN <= numel) {
        const int64_t byte0 = e0 * ES;
        uint32_t lane_off[U];
        float acc[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lane_off[u] = (u * BLOCK + threadIdx.x) * 16u;
            // (kept as they are, so that the second vector's loads take the base + offset form too, not 64-bit additions)
            if (OUT == OUT_BINARY32 || (OUT == OUT_GRAD && FORM != 1)) asm volatile("" : "+v"(lane_off[u]));
        }
        if constexpr (OUT == OUT_FLAT) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[u][i] = -0.0f;
            char* const place = slot + byte0;
            void* const* __restrict__ const rows = t.grad + static_cast<int64_t>(g) * t.R;
            int r = 0;
            for (; r + 8 <= R; r += 8) chunk_copy<DT, NT, 8, U>(rows, r, used, byte0, place + r * flat.stride, flat.stride, lane_off, acc);
            if (r + 4 <= R) { chunk_copy<DT, NT, 4, U>(rows, r, used, byte0, place + r * flat.stride, flat.stride, lane_off, acc); r += 4; }
            if (r + 2 <= R) { chunk_copy<DT, NT, 2, U>(rows, r, used, byte0, place + r * flat.stride, flat.stride, lane_off, acc); r += 2; }
            if (r < R) chunk_copy<DT, NT, 1, U>(rows, r, used, byte0, place + r * flat.stride, flat.stride, lane_off, acc);
            // the averaged bucket is read again by the write-back
#pragma unroll
            for (int u = 0; u < U; ++u) store16(place + R * flat.stride + lane_off[u], scaled<DT>(sc, acc[u]));
            return;
        }
        if (all_used)
            sum_interior_pre<DT, NT, U>(
                pre, byte0, [&](int r) {
                    if constexpr (FORM == 2) return static_cast<const char*>(t.grad[static_cast<int64_t>(g) * t.R + r]) + byte0;
                    else return static_cast<const char*>(row[r]) + byte0;
                }, R, lane_off, acc);
        else if constexpr (MASKED)
            sum_interior_used<DT, NT, U>(row, byte0, used, lane_off, acc);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (OUT == OUT_BINARY32) {
                float y[VEC];
#pragma unroll
                for (int i = 0; i < VEC; ++i) y[i] = apply_scale(sc, acc[u][i]);
                if constexpr (OUT == OUT_BINARY32) store_out32_wave<DT, NT>(outp, byte0 + lane_off[u], y);
                continue;
            }
            const u32x4 out = scaled<DT>(sc, acc[u]);
            store16s<NT>(const_cast<char*>(pre[0]) + byte0 + lane_off[u], out);
            for (int w = 1; w < nwrite; ++w)
                store16u<NT>(row[w] + byte0 + lane_off[u], out);
        }
        return;
    }

    if (e0 >= numel) return;
    // The ends of the segment, element by element: sixteen threads to a replica fetch them ahead of the
    // vectors, all replicas at once, and put them side by side in LDS behind those, where they are summed in
    // ascending order.  When the lane that owned such a vector fetched its elements itself, behind the
    // vectors and eight replicas at a time, a launch of 128 tiles with two tensors took, bfloat16, R = 8 10.6 us
    // and 6.1 so, R = 24 25 and 12, R = 64 60 and 26; binary32 R = 24 14.2 and 11.6, R = 64 33 and 26.
    const EdgeElements ed = edge_elements<VEC>(e0, SPAN, numel);
    const int nedge = ed.head + ed.tail;
    const int slot_k = threadIdx.x % EDGE_SLOTS, slot_r = threadIdx.x / EDGE_SLOTS;
    const int64_t edge_el = slot_k < ed.head ? slot_k : ed.last + (slot_k - ed.head);
    constexpr int EDGE_LOADS = MAX_REPLICAS * EDGE_SLOTS / BLOCK;
    bits edge_x[EDGE_LOADS];
    if (!zero && slot_k < nedge) {
#pragma unroll
        for (int i = 0; i < EDGE_LOADS; ++i) {
            const int r = slot_r + i * (BLOCK / EDGE_SLOTS);
            edge_x[i] = 0;
            if (r < R && ((used >> r) & 1u)) edge_x[i] = gload<bits>(row[r] + edge_el * ES);
        }
    }
    {
        int64_t off[U];
        bool full[U], ok[U];
        float acc[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = e0 + static_cast<int64_t>(u * BLOCK + threadIdx.x) * VEC;
            full[u] = e >= 0 && e + VEC <= numel;
            ok[u] = full[u] && !zero;
            off[u] = e * ES;
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[u][i] = -0.0f;
        }
        if (!zero) {
            // vectors sit on replica 0's 16-byte grid; replicas that are shifted against it
            // are read with element-aligned 16-byte loads
            // (flat buckets: vectors sit on the slot's grid)
            const bool aligned = OUT != OUT_FLAT && src_aligned;
            int r = 0;
            for (; r + 8 <= R; r += 8) chunk_seg<DT, NT, 8, U>(row, r, used, aligned, off, ok, acc, slot, flat.stride);
            if (r + 4 <= R) { chunk_seg<DT, NT, 4, U>(row, r, used, aligned, off, ok, acc, slot, flat.stride); r += 4; }
            if (r + 2 <= R) { chunk_seg<DT, NT, 2, U>(row, r, used, aligned, off, ok, acc, slot, flat.stride); r += 2; }
            if (r < R) { chunk_seg<DT, NT, 1, U>(row, r, used, aligned, off, ok, acc, slot, flat.stride); }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!full[u]) continue;
            float y[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) y[i] = zero ? 0.0f : apply_scale(sc, acc[u][i]);
            if (OUT == OUT_BINARY32) {
                if constexpr (OUT == OUT_BINARY32) store_out32<DT, NT>(outp, off[u], y, si.out_congruent());
                continue;
            }
            if (OUT == OUT_FLAT) {
                store16(slot + R * flat.stride + off[u], Fmt<DT>::narrow(y));
                continue;
            }
            const u32x4 out = zero ? zero16() : Fmt<DT>::narrow(y);
            store16s<NT>(row[0] + off[u], out);
            for (int w = 1; w < nwrite; ++w) {
                char* d = row[w];
                if (src_aligned) store16s<NT>(d + off[u], out);
                else store16u<NT>(d + off[u], out);
            }
        }
    }
    if (nedge == 0) return;
    if (!zero && slot_k < nedge) {
#pragma unroll
        for (int i = 0; i < EDGE_LOADS; ++i) {
            const int r = slot_r + i * (BLOCK / EDGE_SLOTS);
            if (r < R) {
                edge[r * EDGE_SLOTS + slot_k] = edge_x[i];
                // (the copy moves bits, not values: a signalling NaN arrives in the bucket as it is)
                if (OUT == OUT_FLAT) gstore<bits>(slot + r * flat.stride + edge_el * ES, edge_x[i]);
            }
        }
    }
    __syncthreads();
    // (every sixteen threads sum the same elements, so that the threads of replica w's write there)
    if (slot_k < nedge && (slot_r == 0 || slot_r < nwrite)) {
        float s = -0.0f;
        if (!zero)
            for (int r = 0; r < R; ++r) s += Fmt<DT>::value(edge[r * EDGE_SLOTS + slot_k]);
        const float y = zero ? 0.0f : apply_scale(sc, s);
        if (OUT == OUT_FLAT) {
            if (slot_r == 0) Fmt<DT>::store1(slot + R * flat.stride + edge_el * ES, y);
        } else if (OUT == OUT_BINARY32) {
            if (slot_r == 0) gstore<float>(outp + edge_el * 4, y);
        } else {
            for (int w = slot_r; w < nwrite; w += BLOCK / EDGE_SLOTS) Fmt<DT>::store1(row[w] + edge_el * ES, y);
        }
    }
}

template <int DT, bool NT, int U, int OUT, typename Masks, int FORM = 0, typename Tables = SegTables>
__global__ __launch_bounds__(BLOCK) void fused_reduce_kernel(Tables t, int64_t tile_base, int R,
                                                             int nwrite, Masks masks, int keep_unused, Scale sc, FlatBuckets flat,
                                                             const GateRecord* __restrict__ gate,
                                                             uint32_t tag, DispatchSignal sig) {
    signal_dispatch(sig);
    fused_tile<DT, NT, U, OUT, Masks, FORM>(t, tile_base + blockIdx.x, R, nwrite, masks, keep_unused, sc, flat, gate, tag);
}

// A short launch.  It has fewer blocks than fill the chip and runs as long as one of them, whose time is the
// chain of its memory accesses: the tables, then a round of loads for every eight replicas, then the ends of
// segments.  So a block owns one slice of a tile here, 1 KiB of every replica (eight times the blocks); its four
// waves fetch C replicas each, all of them under way at once, and meet in LDS, where thread i sums dword i of
// the slice over the replicas in ascending order.  (C: R / 4, rounded up, at most.)
// The kernel alone, us, a tile per block / slices: one tile of two tensors, bfloat16, R = 24 19 / 4.1, R = 64 44 / 5.7
// (before the ends of segments were fetched together), sixty tensors, 64 tiles, binary32 R = 8 4.6 / 4.1, R = 32 9.8 / 6.2,
// R = 64 17.5 / 12.1, bfloat16 R = 8 5.6 / 4.4, R = 16 7.8 / 5.7, R = 64 20.7 / 13.7.
// Per byte a slice costs more than a tile (a whole wave per KiB of a replica, 4-byte stores): slice_tiles() has
// the line.  Half as long slices, two replicas per load instruction, took three times as long.
template <int DT, int C, int OUT, typename Masks, typename Tables = SegTables>
__global__ __launch_bounds__(BLOCK) void slice_reduce_kernel(Tables t, int64_t base, int R, int nwrite,
                                                             Masks masks, int keep_unused, Scale sc, FlatBuckets flat,
                                                             const GateRecord* __restrict__ gate, uint32_t tag,
                                                             DispatchSignal sig) {
    constexpr int ES = Fmt<DT>::ES;
    constexpr int VEC = Fmt<DT>::VEC;
    constexpr int WORDS = SLICE_BYTES / 4;          // dwords of a slice, one per thread
    constexpr int EPW = 4 / ES;                     // elements of a dword
    typedef typename std::conditional<ES == 4, uint32_t, uint16_t>::type bits;
    static_assert(WORDS == BLOCK && SLICE_BYTES == 64 * 16, "one dword per thread, one vector per lane");
    extern __shared__ __align__(16) uint32_t shared_words[];
    uint32_t* const gathered = shared_words;       // [R][WORDS]
    signal_dispatch(sig);
    const uint32_t gate_word = gate != nullptr ? cload(&gate->failed_tag) : ~tag;
    const int64_t slice = slice_of(t, base, static_cast<int>(blockIdx.x)), tile = slice / SLICES;
    const int g = segment_of(t, tile);
    const auto row = gradients_of(t, g);
    const SegInfo si = segment(t, g);
    const bool masked = masks.present();
    const uint64_t mask = masked ? masks.of(g) : 0;
    if (gate_word == tag) return;
    const int64_t numel = si.numel;
    const int sh = (OUT == OUT_FLAT ? static_cast<int>(si.flat_byte & 15) : si.lead_bytes()) / ES;
    // the slice holds the elements [e0, e0 + SLICE_BYTES / ES) as far as they exist
    const int64_t e0 = (tile - si.tile0) * (TILE_BYTES / ES) + static_cast<int>(slice % SLICES) * (SLICE_BYTES / ES) - sh;
    if (e0 >= numel) return;
    const uint64_t everyone = R >= 64 ? ~uint64_t(0) : ((uint64_t(1) << R) - 1);
    const uint64_t used = masked ? mask : everyone;
    if (OUT != OUT_FLAT && used == 0 && keep_unused) return;
    char* const slot = OUT == OUT_FLAT ? flat.slab0 + si.flat_byte : nullptr;
    // the ends of the segment, element by element, sixteen threads to a replica
    const EdgeElements ed = edge_elements<VEC>(e0, SLICE_BYTES / ES, numel);
    const int nedge = ed.head + ed.tail;
    const int slot_k = threadIdx.x % EDGE_SLOTS, slot_r = threadIdx.x / EDGE_SLOTS;
    const int64_t edge_el = slot_k < ed.head ? slot_k : ed.last + (slot_k - ed.head);
    bits edge_x[C / 4];
    if (slot_k < nedge) {
#pragma unroll
        for (int i = 0; i < C / 4; ++i) {
            const int r = slot_r + i * (BLOCK / EDGE_SLOTS);
            edge_x[i] = 0;
            if (r < R && ((used >> r) & 1u)) edge_x[i] = gload<bits>(row[r] + edge_el * ES);
        }
    }
    {
        // wave w takes Q consecutive replicas; their pointers come in one or two scalar loads (which may reach
        // into the padding behind the table), and all Q loads are issued before the first is waited for
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
        const int Q = (R + 3) / 4, first = wave * Q, count = min(Q, R - first);
        const int64_t e = e0 + lane * VEC;
        const bool full = e >= 0 && e + VEC <= numel;
        const int64_t off = e * ES;
        if (count > 0) {
            const char* base[C];
#pragma unroll
            for (int i = 0; i < C; ++i) base[i] = row[first + i];
            u32x4 x[C];
#pragma unroll
            for (int i = 0; i < C; ++i) {
                x[i] = zero16();
                if (i < count && ((used >> (first + i)) & 1u) && full) x[i] = load16u<true>(base[i] + off);
            }
#pragma unroll
            for (int i = 0; i < C; ++i) {
                if (i < count && full) {
                    *reinterpret_cast<u32x4*>(&gathered[(first + i) * WORDS + lane * 4]) = x[i];
                    if (OUT == OUT_FLAT) store16s<true>(slot + (first + i) * flat.stride + off, x[i]);
                }
            }
        }
    }
    if (slot_k < nedge) {
#pragma unroll
        for (int i = 0; i < C / 4; ++i) {
            const int r = slot_r + i * (BLOCK / EDGE_SLOTS);
            if (r < R) {
                reinterpret_cast<bits*>(gathered)[r * (SLICE_BYTES / ES) + static_cast<int>(edge_el - e0)] = edge_x[i];
                if (OUT == OUT_FLAT) gstore<bits>(slot + r * flat.stride + edge_el * ES, edge_x[i]);
            }
        }
    }
    __syncthreads();
    float acc[EPW];
#pragma unroll
    for (int k = 0; k < EPW; ++k) acc[k] = -0.0f;
    int r = 0;
    for (; r + 8 <= R; r += 8) {
        uint32_t w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = gathered[(r + i) * WORDS + threadIdx.x];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int k = 0; k < EPW; ++k) acc[k] += Fmt<DT>::value(EPW == 1 ? w[i] : k == 0 ? w[i] & 0xFFFFu : w[i] >> 16);
    }
    for (; r < R; ++r) {
        const uint32_t w = gathered[r * WORDS + threadIdx.x];
#pragma unroll
        for (int k = 0; k < EPW; ++k) acc[k] += Fmt<DT>::value(EPW == 1 ? w : k == 0 ? w & 0xFFFFu : w >> 16);
    }
    const bool zero = OUT != OUT_FLAT && used == 0;
    const int64_t e = e0 + static_cast<int>(threadIdx.x) * EPW;
    float y[EPW];
    bool in[EPW];
    bool all = true;
#pragma unroll
    for (int k = 0; k < EPW; ++k) {
        y[k] = zero ? 0.0f : apply_scale(sc, acc[k]);
        in[k] = e + k >= 0 && e + k < numel;
        all = all && in[k];
    }
    if constexpr (OUT == OUT_BINARY32) {
        char* const out = pointer_row(t.out, g, 1)[0];
#pragma unroll
        for (int k = 0; k < EPW; ++k)
            if (in[k]) gstore<float>(out + (e + k) * 4, y[k]);
        return;
    }
    uint32_t word = 0;
    if constexpr (ES == 4) word = __float_as_uint(y[0]);
    else word = Fmt<DT>::down(y[0]) | (Fmt<DT>::down(y[EPW - 1]) << 16);
    const int writes = OUT == OUT_FLAT ? 1 : nwrite;
    for (int w = 0; w < writes; ++w) {
        char* const out = (OUT == OUT_FLAT ? slot + R * flat.stride : row[w]) + e * ES;
        if (all) {
            gstore<u32_a2>(out, word);
        } else {
#pragma unroll
            for (int k = 0; k < EPW; ++k)
                if (in[k]) gstore<bits>(out + k * ES, static_cast<bits>(k == 0 ? word : word >> 16));
        }
    }
}

// ---- stream ordering through device flags ------------------------------------
constexpr uint32_t MAX_GATE_POLLS = 1u << 22;

// Memory ordering of the handshake.  What the bucket kernel must see is written
// by kernels that precede the announcement on the backward stream, and the bucket
// kernel is a launch of its own behind the gate.  Both hops are kernel boundaries
// of a stream: the writers have ended (their results are released to the device)
// before the announcing kernel starts, and the bucket kernel acquires at its
// start, after the gate has ended.  The sequence number itself therefore needs no
// release or acquire of its own -- a release here would only write back this
// XCD's L2, which holds none of the gradients in question but a good deal of the
// concurrently running reduce kernel's lines (measured: 11 us per announcement
// next to a BERT-sized reduction) -- just device-wide atomicity and visibility,
// which relaxed agent-scope atomics give.
// host: pinned word that receives the number too, or null.
__global__ __launch_bounds__(64) void announce_kernel(OrderState* st, unsigned long long seq, unsigned long long* host) {
    if (threadIdx.x == 0) {
        __hip_atomic_store(&st->ready_seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (host != nullptr) __hip_atomic_store(host, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// One wave; lane 0 polls.  Both bounds (wall-clock ticks and the poll count) end
// the loop whatever the other stream does.
__global__ __launch_bounds__(64) void gate_kernel(OrderState* st, unsigned long long need,
                                                  long long wait_ticks, GateRecord* rec, GateRecord* row_summary,
                                                  int32_t tile_base, int32_t ntiles, int32_t dtype,
                                                  uint32_t tag, unsigned long long chain_ord, long long chain_ticks) {
    if (threadIdx.x != 0) return;
    bool ok = false;
    if (__hip_atomic_load(&st->abort_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != tag) {
        const uint64_t t0 = wall_clock64();
        for (uint32_t poll = 0; poll < MAX_GATE_POLLS; ++poll) {
            if (__hip_atomic_load(&st->ready_seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= need) {
                ok = true;
                break;
            }
            if (static_cast<long long>(wall_clock64() - t0) >= wait_ticks) break;
            __builtin_amdgcn_s_sleep(2);
        }
    }
    if (ok && chain_ticks > 0) {
        // scheduling only: let the launch this one is chained to reach its last block first
        const uint64_t t1 = wall_clock64();
        for (uint32_t poll = 0; poll < MAX_GATE_POLLS; ++poll) {
            if (__hip_atomic_load(&st->dispatched, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= chain_ord) break;
            if (static_cast<long long>(wall_clock64() - t1) >= chain_ticks) break;
            __builtin_amdgcn_s_sleep(2);
        }
    }
    if (!ok) {
        rec->tile_base = tile_base;
        rec->ntiles = ntiles;
        rec->dtype = dtype;
        rec->failed_tag = tag;
        row_summary->failed_tag = tag;
        __hip_atomic_store(&st->abort_tag, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The same handshake in the other direction, once per iteration and reduction stream: the stream's bucket
// kernels have ended, and their results are released, when done_kernel runs, and what follows the wait for the
// number on the backward stream starts after it.
__global__ __launch_bounds__(64) void done_kernel(unsigned long long* word, unsigned long long tag) {
    if (threadIdx.x == 0) __hip_atomic_store(word, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(64) void chain_wait_kernel(OrderState* st, unsigned long long chain_ord, long long chain_ticks) {
    if (threadIdx.x != 0) return;
    const uint64_t t0 = wall_clock64();
    for (uint32_t poll = 0; poll < MAX_GATE_POLLS; ++poll) {
        if (__hip_atomic_load(&st->dispatched, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= chain_ord) break;
        if (static_cast<long long>(wall_clock64() - t0) >= chain_ticks) break;
        __builtin_amdgcn_s_sleep(2);
    }
}

// Launches whose gate gave up, redone once every gradient exists.  Block j takes
// the tiles j, j + G, ... of each failed launch.
template <int DT, bool NT, int U, int OUT>
__global__ __launch_bounds__(BLOCK) void repair_kernel(SegTables t, OrderState* st,
                                                       const GateRecord* __restrict__ rec,
                                                       int nb, uint32_t tag, int R, int nwrite,
                                                       const uint64_t* __restrict__ local,
                                                       int keep_unused, Scale sc, FlatBuckets flat) {
    // rec[nb] is the row's summary: no gate of the iteration gave up (the normal case), nothing to look for
    if (rec[nb].failed_tag != tag) return;
    for (int b = 0; b < nb; ++b) {
        const GateRecord r = rec[b];
        if (r.failed_tag != tag || r.dtype != DT) continue;
        if (blockIdx.x == 0 && threadIdx.x == 0) st->repaired += 1;   // (repair launches run one after the other)
        for (int64_t i = blockIdx.x; i < r.ntiles; i += gridDim.x) {
            __syncthreads();       // the tile before is done with its elements in LDS
            fused_tile<DT, NT, U, OUT>(t, r.tile_base + i, R, nwrite, MaskTable{local}, keep_unused, sc, flat);
        }
    }
}

// Whether *word became `value` within `ticks`.
__device__ __forceinline__ bool poll_for(unsigned long long* word, unsigned long long value, long long ticks) {
    const uint64_t t0 = wall_clock64();
    for (uint32_t poll = 0; poll < MAX_GATE_POLLS; ++poll) {
        if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == value) return true;
        if (static_cast<long long>(wall_clock64() - t0) >= ticks) break;
        __builtin_amdgcn_s_sleep(16);
    }
    return false;
}

__global__ __launch_bounds__(64) void probe_wait_kernel(unsigned long long* word, unsigned long long value, long long wait_ticks) {
    if (threadIdx.x != 0) return;
    __hip_atomic_store(&word[2], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word[1] = poll_for(&word[0], value, wait_ticks) ? 1 : 0;
}

__global__ __launch_bounds__(64) void probe_write_kernel(unsigned long long* word, unsigned long long value, long long wait_ticks) {
    if (threadIdx.x == 0 && poll_for(&word[2], value, wait_ticks))
        __hip_atomic_store(&word[0], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- K4: no_sync accumulation ---------------------------------------------
// a + b, elementwise, rounded to storage
template <int DT>
__device__ __forceinline__ u32x4 added(u32x4 a, u32x4 b) {
    float fa[Fmt<DT>::VEC], fb[Fmt<DT>::VEC];
    Fmt<DT>::widen(a, fa);
    Fmt<DT>::widen(b, fb);
#pragma unroll
    for (int i = 0; i < Fmt<DT>::VEC; ++i) fa[i] = fa[i] + fb[i];
    return Fmt<DT>::narrow(fa);
}

// Bound by HBM: two reads and one write of every byte.
// STREAM: the gradients' loads and stores carry the non-temporal hint as the micro-step's loads always
// do (launch_accumulate has the rule).  Two vectors per thread; one or four vectors and replicas in turn block by block were
// no better.  Three to six resident blocks (auto_accumulate_blocks in the host code).
template <int DT, bool STREAM>
__device__ __forceinline__ void accumulate_tile(const char* __restrict__ src, char* dst,
                                                int64_t numel, int64_t ltile) {
    constexpr int ES = Fmt<DT>::ES;
    constexpr int VEC = Fmt<DT>::VEC;
    constexpr int U = 2;
    const int sh = lead_in(dst, ES);
    const int64_t e_tile = ltile * (TILE_BYTES / ES) - sh;
    if (e_tile >= 0 && e_tile + TILE_BYTES / ES <= numel) {
        // the whole tile is inside the segment: no lane is predicated, offsets are 32 bits
        src += e_tile * ES;
        dst += e_tile * ES;
#pragma unroll 1
        for (int step = 0; step < TILE_VECS / (BLOCK * U); ++step) {
            u32x4 a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t off = ((step * U + u) * BLOCK + threadIdx.x) * 16u;
                a[u] = load16<STREAM>(dst + off);
                b[u] = load16u<true>(src + off);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                store16s<STREAM>(dst + ((step * U + u) * BLOCK + threadIdx.x) * 16u, added<DT>(a[u], b[u]));
        }
        return;
    }
#pragma unroll 1
    for (int step = 0; step < TILE_VECS / (BLOCK * U); ++step) {
        int64_t e[U];
        int kind[U];
        u32x4 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            e[u] = e_tile + static_cast<int64_t>((step * U + u) * BLOCK + threadIdx.x) * VEC;
            kind[u] = classify(e[u], VEC, numel);
            a[u] = zero16();
            b[u] = zero16();
            if (kind[u] == V_FULL) {
                a[u] = load16<STREAM>(dst + e[u] * ES);
                b[u] = load16u<true>(src + e[u] * ES);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kind[u] == V_FULL) {
                store16s<STREAM>(dst + e[u] * ES, added<DT>(a[u], b[u]));
            } else if (kind[u] == V_EDGE) {
                for (int i = 0; i < VEC; ++i) {
                    const int64_t idx = e[u] + i;
                    if (idx < 0 || idx >= numel) continue;
                    const float s = Fmt<DT>::load1(dst + idx * ES) + Fmt<DT>::load1(src + idx * ES);
                    Fmt<DT>::store1(dst + idx * ES, s);
                }
            }
        }
    }
}

// Where a block finds its micro-gradient: in a table in device memory, or in the launch's arguments.
struct MicroTable {
    void* const* row0;
    __device__ __forceinline__ const char* operator()(int g, int r, int R) const { return pointer_row(row0, g, R)[r]; }
};
// The arguments save the kernel that brings a table to the device and its hand-over, 4.7 us of the stream, and one of two launches
// of the host; 512 bytes of them cost the host no more than none, 3.5 KiB 1.4 us.  Us a micro-step, table / arguments:
// R = 2, four tensors 6.7 / 4.2, R = 8, forty 11.2 / 8.4, R = 4, 175 16.2 / 13.6, R = 16, 87 24.4 / 22.5 (all bound by the list's way
// through Python); four micro-steps and the reduction, R = 8, sixty tensors 57.6 / 48.3, R = 16, 200 tensors of 10 MB 328 / 314; ResNet-50
// in bfloat16, R = 8 194.0 / 192.7.
template <int N>
struct MicroWords {
    uint64_t w[N];
    int32_t regular;           // w: R bases and a distance for each segment; else the table itself
    __device__ __forceinline__ const char* operator()(int g, int r, int R) const {
        const uint64_t a = regular ? w[r] : 0, d = regular ? w[R + g] : w[g * R + r];
        return d == kMicroAbsent ? nullptr : reinterpret_cast<const char*>(a + d);
    }
};

template <bool STREAM, typename Micro>
__global__ __launch_bounds__(BLOCK) void accumulate_kernel(SegTables t, Micro micro) {
    const int64_t tile = blockIdx.x;
    const int r = blockIdx.y;
    const int g = cload(t.tile_seg + tile);
    const SegInfo si = segment(t, g);
    const char* src = micro(g, r, t.R);
    char* dst = pointer_row(t.grad, g, t.R)[r];
    if (src == nullptr) return;
    const int64_t numel = si.numel;
    const int64_t ltile = tile - si.tile0;
    switch (si.dtype()) {
        case 0: accumulate_tile<0, STREAM>(src, dst, numel, ltile); break;
        case 1: accumulate_tile<1, STREAM>(src, dst, numel, ltile); break;
        default: accumulate_tile<2, STREAM>(src, dst, numel, ltile); break;
    }
}

// The pointers of a micro-step go from pinned memory to the table that accumulate_kernel reads, and `done`
// (pinned) tells the host with which call's it is through, so that the host may write there again.  The last of a block's
// reads has returned when its threads have met, so neither the count of blocks that are through (`arrived`, 0 between
// launches) nor the store needs a release (which would write the cache back).  Bound by the way to host memory and back, about
// 2 us; every thread keeps four 16-byte loads under way, a block takes 64 KiB a round, and a table takes as many blocks, up to 32.
// A copy of the runtime's and an event behind it took 2.9 and 4 us of the host, the wait for the event 7 when it had
// just passed, and 10 us of the stream: ResNet-50 in bfloat16, R = 8, 196 -> 193 us a micro-step; 234 tensors, R = 5, 57 -> 50;
// four micro-steps and the reduction of 84000 elements, R = 16, 270 -> 239.  Large tables (pointers ready in an array, us a micro-step, the
// runtime's copy / one block / so): R = 64, 2000 tensors 401 / 447 / 379, 8000 1662 / 1851 / 1622; R = 32, 1600 tensors 521 / 533 / 511 (the
// kernel alone 40 / 12).
// MANY: more than one block.  (A table that one block takes is spared the count: R = 2, four tensors, 6.2 us a micro-step, 7.8 with it.)
constexpr int POINTER_COPY_LOADS = 4, POINTER_COPY_BLOCKS = 32;
template <bool MANY>
__global__ __launch_bounds__(1024) void pointer_copy_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src, int64_t nvec, int blocks,
                                                            unsigned* arrived, unsigned long long* done, unsigned long long ticket) {
    constexpr int U = POINTER_COPY_LOADS;
    for (int64_t i0 = (MANY ? static_cast<int64_t>(blockIdx.x) * 1024 * U : 0) + threadIdx.x; i0 < nvec;
         i0 += static_cast<int64_t>(MANY ? blocks : 1) * 1024 * U) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * 1024 < nvec) v[u] = src[i0 + u * 1024];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * 1024 < nvec) dst[i0 + u * 1024] = v[u];
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (MANY) {
        if (__hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 < static_cast<unsigned>(blocks)) return;
        __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __hip_atomic_store(done, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- global participation bitmap ---------------------------------------------
// Up to kMasksByValue masks reach the device inside kernel arguments instead of by
// a staged copy, which takes the host three times as long and the stream a copy packet with a hand-over
// on each side.  ResNet-50, R = 8, 0.7 of the flags set, one mark per call: 502 us a synchronization
// with copies, flag bytes, the predicated path for every such tile and marks that pass a numpy array
// through ctypes; 149 us with masks, sum_interior_used and marks in C.
struct MaskPayload {
    uint64_t m[kMasksByValue];
    __device__ __forceinline__ uint64_t of(int i) const { return m[i]; }
};

// More are read from pinned memory, by one launch whatever their number.  A tenth of the parameters
// never marked, R = 4, all marks in one call, us a synchronization with staged copies / a launch of
// arguments for every 384 masks / pinned memory: 500 parameters 51 / 38 / 25, 1000 61 / 50 / 33,
// 4000 114 / 155 / 82, 20000 404 / 683 / 345.  (Pinned memory for fewer than 384 is no faster than
// arguments, 24 / 24, and has the host wait for the iteration before the last.)
struct MaskPointer {
    const uint64_t* m;
    __device__ __forceinline__ uint64_t of(int i) const { return m[i]; }
};

// rows [0, count) of one launch; a launch whose gate gave up reads no masks, and its rows may still
// be read by the previous iteration's repair launch
template <typename Masks>
__global__ __launch_bounds__(BLOCK) void mask_write_kernel(uint64_t* __restrict__ dst, Masks p, int count,
                                                           const GateRecord* __restrict__ gate, uint32_t tag) {
    if (gate != nullptr && gate->failed_tag == tag) return;
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    if (i < count) dst[i] = p.of(i);
}

// The one-GPU form of the extra AllReduce on the unused-parameter bitmap
// (Section 4.2): global[g] = OR over the R replicas of bit r of local[g], for the device (write-back)
// and for the host (pinned memory; a word tells by itself whose iteration's it is).
template <typename Masks>
__global__ __launch_bounds__(BLOCK) void bitmap_or_kernel(uint64_t* __restrict__ local, uint8_t* __restrict__ global,
                                                          uint64_t* __restrict__ host_global, uint64_t tag, Masks p, int count) {
    const int g = blockIdx.x * BLOCK + threadIdx.x;
    if (g >= count) return;
    const uint64_t mask = p.of(g);
    const uint8_t any = mask != 0 ? 1 : 0;
    local[g] = mask;
    global[g] = any;
    __hip_atomic_store(host_global + g, tag * 2 + any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- K6: synthetic backward emitter -----------------------------------------
// With ticks > 0 every wave waits until `ticks` of the constant-rate wall clock
// have passed (at most MAX_SPINS polls, so the kernel always ends); with a
// pointer row replica blockIdx.y's gradient is copied from its source.  The
// host launches the two roles separately (launch_emit).
constexpr uint32_t MAX_SPINS = 1u << 20;

__global__ __launch_bounds__(BLOCK) void emit_kernel(int64_t ticks, void* const* __restrict__ ptrs,
                                                     int R, int64_t nelem, int es, int busy,
                                                     float* __restrict__ sink) {
    if (ticks > 0) {
        const uint64_t t0 = wall_clock64();
        float a = static_cast<float>(threadIdx.x);
        for (uint32_t spin = 0; spin < MAX_SPINS; ++spin) {
            if (static_cast<int64_t>(wall_clock64() - t0) >= ticks) break;
            if (busy) {
                // arithmetic between polls: the delay looks like compute to the GPU's
                // power management instead of like an idle wait
#pragma unroll
                for (int i = 0; i < 64; ++i) a = a * 1.0000001f + 0.5f;
            } else {
                __builtin_amdgcn_s_sleep(4);
            }
        }
        if (busy && a == 12345.678f && sink != nullptr) sink[0] = a;   // keeps the arithmetic alive
    }
    if (ptrs == nullptr) return;
    const int r = blockIdx.y;
    if (r >= R) return;
    char* dst = static_cast<char*>(ptrs[r]);
    const char* src = static_cast<const char*>(ptrs[R + r]);
    const int64_t stride = static_cast<int64_t>(gridDim.x) * BLOCK;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * BLOCK + threadIdx.x; i < nelem; i += stride) {
        if (es == 4) gstore<uint32_t>(dst + i * 4, gload<uint32_t>(src + i * 4));
        else gstore<uint16_t>(dst + i * 2, gload<uint16_t>(src + i * 2));
    }
}

inline hipError_t after_launch() { return hipGetLastError(); }

// Every kernel here streams through HBM and needs only a few resident blocks per
// CU to keep the memory system full; more blocks mean more interleaved request
// streams at the DRAM channels and measurably less throughput.  `lds` bytes of
// dynamic LDS cap the number of resident blocks (a CU has 160 KiB of LDS): 0 = no cap.  For the kernels that keep
// data there it is a required minimum, too: edge_lds(R) for whole tiles and repairs, R * SLICE_BYTES for slices.
constexpr unsigned kLdsNoOptIn = 64 * 1024;
constexpr unsigned kLdsPerUnit = 160 * 1024;     // gfx950

// the pair of events that the next launch through launch() on this thread carries (time_next_launch)
thread_local hipEvent_t g_time_start = nullptr, g_time_stop = nullptr;

template <typename... KArgs, typename... Args>
static hipError_t launch(void (*kernel)(KArgs...), dim3 grid, unsigned lds, hipStream_t s, const Args&... args) {
    if (lds > kLdsNoOptIn) {
        // allocations above 64 KiB must be allowed per kernel; once is enough
        // (per device: the attribute belongs to the kernel's code object on the current device)
        static std::mutex mu;
        static std::set<std::pair<int, const void*>> raised;
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const std::pair<int, const void*> key(dev, reinterpret_cast<const void*>(kernel));
        std::lock_guard<std::mutex> lock(mu);
        if (raised.find(key) == raised.end()) {
            e = hipFuncSetAttribute(key.second, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    static_cast<int>(kLdsPerUnit));
            if (e != hipSuccess) return e;
            raised.insert(key);
        }
    }
    if (g_time_start) {
        // the runtime stamps the two events with this kernel's own start and end: no packet of
        // its own sits between consecutive kernels, as an event record would
        hipEvent_t a = g_time_start, b = g_time_stop;
        g_time_start = g_time_stop = nullptr;
        hipExtLaunchKernelGGL(kernel, grid, dim3(BLOCK), lds, s, a, b, 0u, static_cast<KArgs>(args)...);
    } else {
        hipLaunchKernelGGL(kernel, grid, dim3(BLOCK), lds, s, static_cast<KArgs>(args)...);
    }
    return hipGetLastError();
}

}  // namespace

// ---- launch wrappers ---------------------------------------------------------
void time_next_launch(hipEvent_t start, hipEvent_t stop) {
    g_time_start = start;
    g_time_stop = stop;
}

bool timing_pair_unused() {
    const bool unused = g_time_start != nullptr;
    g_time_start = g_time_stop = nullptr;
    return unused;
}

hipError_t launch_pack(const SegTables& t, int64_t tile_base, int64_t ntiles, char* slab0,
                       int64_t slab_stride, int nrep, const uint64_t* local,
                       const GateRecord* gate, uint32_t tag, hipStream_t s) {
    if (ntiles <= 0 || nrep <= 0) return hipSuccess;
    dim3 grid(static_cast<unsigned>(ntiles), static_cast<unsigned>(nrep));
    return launch(gate != nullptr ? seg_copy_kernel<true, true> : seg_copy_kernel<true, false>, grid, 0u, s, t, tile_base, slab0, slab_stride, local, nullptr, 0, gate, tag);
}

hipError_t launch_unpack(const SegTables& t, int64_t tile_base, int64_t ntiles,
                         const char* out_slab, int nrep, const uint8_t* global_used, bool keep_unused,
                         hipStream_t s) {
    if (ntiles <= 0 || nrep <= 0) return hipSuccess;
    dim3 grid(static_cast<unsigned>(ntiles), static_cast<unsigned>(nrep));
    const int keep = keep_unused ? 1 : 0;
    return launch(seg_copy_kernel<false, false>, grid, 0u, s, t, tile_base, const_cast<char*>(out_slab), int64_t(0), nullptr, global_used, keep, nullptr, 0u);
}

// Vectors per thread and replica in the reduce kernels: a tile's worth (two), which measured
// best against one and four on both model-shaped lists.
constexpr int RU = TILE_VECS / BLOCK;

template <int DT>
static hipError_t flat_reduce_dispatch(bool nt, unsigned lds, hipStream_t s, const char* in0, int64_t stride,
                                       char* out, int64_t nvec, int R, Scale sc,
                                       const GateRecord* gate, uint32_t tag, DispatchSignal sig) {
    const int64_t nrows = (nvec + BLOCK * RU - 1) / (BLOCK * RU);
    dim3 grid(static_cast<unsigned>(nrows));
    const bool gated = gate != nullptr || sig.word != nullptr;
    if (nt) return launch(gated ? flat_reduce_kernel<DT, true, RU, true> : flat_reduce_kernel<DT, true, RU, false>, grid, lds, s, in0, stride, out, nvec, R, sc, gate, tag, sig);
    return launch(gated ? flat_reduce_kernel<DT, false, RU, true> : flat_reduce_kernel<DT, false, RU, false>, grid, lds, s, in0, stride, out, nvec, R, sc, gate, tag, sig);
}

hipError_t launch_flat_reduce(int dtype, const char* in0, int64_t stride, char* out, int64_t nvec,
                              int R, Scale sc, bool nontemporal, unsigned lds,
                              const GateRecord* gate, uint32_t tag, DispatchSignal sig, hipStream_t s) {
    if (nvec <= 0) return hipSuccess;
    switch (dtype) {
        case 0: return flat_reduce_dispatch<0>(nontemporal, lds, s, in0, stride, out, nvec, R, sc, gate, tag, sig);
        case 1: return flat_reduce_dispatch<1>(nontemporal, lds, s, in0, stride, out, nvec, R, sc, gate, tag, sig);
        case 2: return flat_reduce_dispatch<2>(nontemporal, lds, s, in0, stride, out, nvec, R, sc, gate, tag, sig);
        default: return hipErrorInvalidValue;
    }
}

// What the ends of segments take (fused_tile).
static unsigned edge_lds(int R) { return static_cast<unsigned>(R * EDGE_SLOTS * sizeof(uint32_t)); }

// How a launch of tiles without masks reads its tables (FORM of fused_tile), which decides when a block's loads go out: whether a
// block's first pointers, its segment and its tile's entry come by scalar or by plain loads, and likewise the pointers of
// replicas 8 and up; and whether the lanes' offsets are kept for the base + offset form.  Long launches are a few percent
// faster with one or the other, see fused_tile, and no form is the best for every R; sixty BERT-large tensors unless noted, us.
// 2: everything plain, from two full rounds of eight replicas on.  One launch, 0 or 1 / 2: binary32 R = 16 835 / 816, R = 24 1259 / 1218, R = 32
// 1658 / 1614 (R = 12 615 / 638, R = 14 726 / 723); bfloat16 R = 16 407 / 398, R = 24 613 / 597, R = 32 806 / 791 (R = 10 255 / 281, R = 12 300 / 316,
// R = 14 354 / 365); binary32 averages R = 16 431 / 427, R = 24 652 / 639, R = 32 858 / 843 (R = 14 379 / 384).  One mark per call, 25 MiB buckets:
// binary32 R = 16 848 / 842, R = 24 1253 / 1243, R = 32 1635 / 1626.
// 1, binary32 averages: first loads plain, further pointers scalar.  2000 MiB, 0 / 1: R = 2 447 / 454, R = 3 424 / 410, R = 4 410 / 390, R = 5 402 /
// 376, R = 6 384 / 394, R = 8 353 / 370, R = 9 355 / 382, R = 10 359 / 368, R = 11 364 / 360 (binary16 317 / 323), R = 14 375 / 360.
// 1, binary32 gradients of which every replica is written: offsets left to the compiler.  2000 MiB, 0 / 1: R = 2 464 / 450, R = 3 506 / 508, R = 4
// 557 / 571, R = 5 583 / 583, R = 6 618 / 600, R = 7 652 / 642, R = 8 682 / 677, R = 10 699 / 670 (25 MiB buckets, one mark per call, 541 / 555), R = 16 742 / 741 (2 is no better).  (One replica
// written, R = 2, 323 / 339; 16 bits, every replica, R = 4 557 / 575.)
// binary16 keeps 0 from sixteen replicas on: its conversions leave the loads of 2 no room (60 tensors, one launch of 4 GB, 0 / 2, R = 16 655 / 720, R = 32
// 656 / 704; with binary32 averages R = 16 672 / 782, R = 32 682 / 829).
// Shorter launches keep 0: there the loads that come sooner count (150 MiB, 0 / 2, binary32 averages, R = 16 29.1 / 29.8, R = 32 32.0 / 33.6; 0 / 1, R = 5
// 31.0 / 31.7; every replica written, R = 64, 67.2 / 68.2; one replica, 470 MiB, R = 24, binary32 80.1 / 81.3, bfloat16 80.9 / 82.3; 950 MiB, 25 MiB buckets, R = 32, 166 / 163
// and 167 / 164).
static int table_form(int dtype, int out, int R, int nwrite, int64_t ntiles) {
    if (ntiles * TILE_BYTES * (R + 1) < (int64_t(600) << 20)) return 0;
    if (R >= 16 && nwrite == 1) return dtype == 1 ? 0 : 2;
    if (out == OUT_BINARY32) return (R >= 3 && R <= 5) || R >= 12 ? 1 : 0;
    return dtype == 0 && nwrite > 1 && (R < 3 || (R > 5 && R <= 8)) ? 1 : 0;
}

template <int DT, int OUT, typename M>
static hipError_t fused_launch(bool nt, int64_t ntiles, unsigned lds, hipStream_t s,
                               const SegTables& t, int64_t tile_base, int R, int nwrite,
                               const M& masks, int keep, Scale sc, FlatBuckets flat,
                               const GateRecord* gate, uint32_t tag, DispatchSignal sig) {
    dim3 grid(static_cast<unsigned>(ntiles));
    lds = std::max(lds, edge_lds(R));
    if constexpr (!M::ANY && OUT != OUT_FLAT) {
        const int form = nt ? table_form(DT, OUT, R, nwrite, ntiles) : 0;
        if constexpr (OUT == OUT_BINARY32 || Fmt<DT>::ES == 4)
            if (form == 1)
                return launch(fused_reduce_kernel<DT, true, RU, OUT, M, 1>, grid, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
        if constexpr (DT != 1)
            if (form == 2)
                return launch(fused_reduce_kernel<DT, true, RU, OUT, M, 2>, grid, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
    }
    if (nt) return launch(fused_reduce_kernel<DT, true, RU, OUT, M>, grid, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
    return launch(fused_reduce_kernel<DT, false, RU, OUT, M>, grid, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
}

template <int DT, int OUT, typename M>
static hipError_t slice_launch(int64_t blocks, hipStream_t s, const SegTables& t, int64_t base, int R, int nwrite,
                               const M& masks, int keep, Scale sc, FlatBuckets flat,
                               const GateRecord* gate, uint32_t tag, DispatchSignal sig) {
    const dim3 grid(static_cast<unsigned>(blocks));
    const unsigned lds = static_cast<unsigned>(R * SLICE_BYTES);
    // (registers and code for sixteen replicas a wave cost 20 % where four will do)
    if (R <= 16) return launch(slice_reduce_kernel<DT, 4, OUT, M>, grid, lds, s, t, base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
    return launch(slice_reduce_kernel<DT, MAX_REPLICAS / 4, OUT, M>, grid, lds, s, t, base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
}

template <int DT, int OUT>
static hipError_t fused_dispatch(bool nt, int64_t ntiles, int64_t slice_base, int64_t nslices, unsigned lds, hipStream_t s,
                                 const SegTables& t, int64_t tile_base, int R, int nwrite,
                                 const Masks& masks, int keep, Scale sc, FlatBuckets flat,
                                 const GateRecord* gate, uint32_t tag, DispatchSignal sig) {
    // (without the hint every launch takes tiles, so that both kernels can be had at any size)
    const bool slices = nt && takes_slices(R, Fmt<DT>::ES, OUT == OUT_FLAT, ntiles, nslices, t.slices != nullptr);
    SegTables ts = t;
    if (!takes_list(R, Fmt<DT>::ES, OUT == OUT_FLAT, ntiles, nslices)) ts.slices = nullptr;
    const int64_t blocks = ts.slices != nullptr ? nslices : ntiles * SLICES, base = ts.slices != nullptr ? slice_base : tile_base;
    auto with = [&](const auto& m) {
        if (slices) return slice_launch<DT, OUT>(blocks, s, ts, base, R, nwrite, m, keep, sc, flat, gate, tag, sig);
        return fused_launch<DT, OUT>(nt, ntiles, lds, s, t, tile_base, R, nwrite, m, keep, sc, flat, gate, tag, sig);
    };
    if (masks.words != nullptr) {
        MaskWords m;
        std::memcpy(m.m, masks.words, sizeof(m.m));
        m.first = masks.first;
        m.shift = mask_shift(R);
        return with(m);
    }
    // (the staged pass reads its masks through chunk_copy's one branch per replica: 329 us with either
    // instance, ResNet-50, R = 8, all marks in one call)
    if (masks.table == nullptr && (OUT != OUT_FLAT || slices)) {
        if constexpr (OUT != OUT_FLAT) return with(NoMasks{});
        else return slice_launch<DT, OUT>(blocks, s, ts, base, R, nwrite, NoMasks{}, keep, sc, flat, gate, tag, sig);
    }
    return with(MaskTable{masks.table});
}

void pack_masks(const uint64_t* masks, int count, int R, uint64_t* words) {
    const int shift = mask_shift(R);
    std::memset(words, 0, sizeof(uint64_t) * kMaskWords);
    for (int k = 0; k < count; ++k) words[(k << shift) >> 6] |= masks[k] << ((k << shift) & 63);
}

hipError_t launch_fused_reduce(int dtype, const SegTables& t, int64_t tile_base, int64_t ntiles, int64_t slice_base, int64_t nslices,
                               int R, int nwrite, const Masks& masks, bool keep_unused, Scale sc,
                               bool nontemporal, unsigned lds, FlatBuckets flat,
                               const GateRecord* gate, uint32_t tag, DispatchSignal sig, hipStream_t s) {
    if (ntiles <= 0) return hipSuccess;
    const int keep = keep_unused ? 1 : 0;
    if (t.out != nullptr) {
        // 16-bit gradients, binary32 averages to separate tensors
        if (nwrite != 1 || flat.slab0 != nullptr) return hipErrorInvalidValue;
        switch (dtype) {
            case 1: return fused_dispatch<1, OUT_BINARY32>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
            case 2: return fused_dispatch<2, OUT_BINARY32>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
            default: return hipErrorInvalidValue;
        }
    }
    if (flat.slab0 != nullptr) {
        switch (dtype) {
            case 0: return fused_dispatch<0, OUT_FLAT>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
            case 1: return fused_dispatch<1, OUT_FLAT>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
            case 2: return fused_dispatch<2, OUT_FLAT>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
            default: return hipErrorInvalidValue;
        }
    }
    switch (dtype) {
        case 0: return fused_dispatch<0, OUT_GRAD>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
        case 1: return fused_dispatch<1, OUT_GRAD>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
        case 2: return fused_dispatch<2, OUT_GRAD>(nontemporal, ntiles, slice_base, nslices, lds, s, t, tile_base, R, nwrite, masks, keep, sc, flat, gate, tag, sig);
        default: return hipErrorInvalidValue;
    }
}

template <int DT, int N>
static hipError_t value_launch(const WordTables& words, int64_t tile_base, int64_t ntiles, int64_t nslices, int R, Scale sc, hipStream_t s) {
    ArgTables<N> t;
    std::memcpy(t.w, words.words, sizeof(uint64_t) * words.count(R));
    t.n = words.n;
    t.R = R;
    t.at = words.n;
    t.step = words.regular ? 0 : R;
    t.dist = words.regular ? words.n + R : 0;
    const FlatBuckets flat{nullptr, 0};
    const DispatchSignal sig{nullptr, 0};
    if (!takes_slices(R, Fmt<DT>::ES, false, ntiles, nslices, false))
        return launch(fused_reduce_kernel<DT, true, RU, OUT_GRAD, NoMasks, 0, ArgTables<N>>, dim3(static_cast<unsigned>(ntiles)), edge_lds(R), s,
                      t, tile_base, R, 1, NoMasks{}, 0, sc, flat, nullptr, 0u, sig);
    const dim3 grid(static_cast<unsigned>(ntiles * SLICES));
    const unsigned lds = static_cast<unsigned>(R * SLICE_BYTES);
    if (R <= 16) return launch(slice_reduce_kernel<DT, 4, OUT_GRAD, NoMasks, ArgTables<N>>, grid, lds, s, t, tile_base, R, 1, NoMasks{}, 0, sc, flat, nullptr, 0u, sig);
    return launch(slice_reduce_kernel<DT, MAX_REPLICAS / 4, OUT_GRAD, NoMasks, ArgTables<N>>, grid, lds, s, t, tile_base, R, 1, NoMasks{}, 0, sc, flat, nullptr, 0u, sig);
}

template <int DT>
static hipError_t value_dispatch(const WordTables& t, int64_t tile_base, int64_t ntiles, int64_t nslices, int R, Scale sc, hipStream_t s) {
    const int64_t count = t.count(R);
    if (count <= 128) return value_launch<DT, 128>(t, tile_base, ntiles, nslices, R, sc, s);
    if (count <= 256) return value_launch<DT, 256>(t, tile_base, ntiles, nslices, R, sc, s);
    return value_launch<DT, kTableWords>(t, tile_base, ntiles, nslices, R, sc, s);
}

hipError_t launch_fused_reduce_by_value(int dtype, const WordTables& t, int64_t tile_base, int64_t ntiles, int64_t nslices, int R, Scale sc,
                                        hipStream_t s) {
    if (ntiles <= 0) return hipSuccess;
    if (t.n <= 0 || R <= 0 || R > MAX_REPLICAS || t.count(R) > kTableWords) return hipErrorInvalidValue;
    switch (dtype) {
        case 0: return value_dispatch<0>(t, tile_base, ntiles, nslices, R, sc, s);
        case 1: return value_dispatch<1>(t, tile_base, ntiles, nslices, R, sc, s);
        case 2: return value_dispatch<2>(t, tile_base, ntiles, nslices, R, sc, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_announce(OrderState* st, unsigned long long seq, unsigned long long* host, hipStream_t s) {
    hipLaunchKernelGGL(announce_kernel, dim3(1), dim3(64), 0, s, st, seq, host);
    return after_launch();
}

hipError_t launch_chain_wait(OrderState* st, unsigned long long chain_ord, long long chain_ticks, hipStream_t s) {
    hipLaunchKernelGGL(chain_wait_kernel, dim3(1), dim3(64), 0, s, st, chain_ord, chain_ticks);
    return after_launch();
}

hipError_t launch_done(unsigned long long* word, unsigned long long tag, hipStream_t s) {
    hipLaunchKernelGGL(done_kernel, dim3(1), dim3(64), 0, s, word, tag);
    return after_launch();
}

hipError_t launch_gate(OrderState* st, unsigned long long need, long long wait_ticks, GateRecord* rec,
                       GateRecord* row_summary, int32_t tile_base, int32_t ntiles, int32_t dtype, uint32_t tag,
                       unsigned long long chain_ord, long long chain_ticks, hipStream_t s) {
    hipLaunchKernelGGL(gate_kernel, dim3(1), dim3(64), 0, s, st, need, wait_ticks, rec, row_summary, tile_base,
                       ntiles, dtype, tag, chain_ord, chain_ticks);
    return after_launch();
}

template <int DT, int OUT>
static hipError_t repair_dispatch(bool nt, int blocks, hipStream_t s, const SegTables& t, OrderState* st,
                                  const GateRecord* rec, int nb, uint32_t tag, int R, int nwrite,
                                  const uint64_t* local, int keep, Scale sc, FlatBuckets flat) {
    const dim3 grid(static_cast<unsigned>(blocks));
    if (nt) return launch(repair_kernel<DT, true, RU, OUT>, grid, edge_lds(R), s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
    return launch(repair_kernel<DT, false, RU, OUT>, grid, edge_lds(R), s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
}

hipError_t launch_repair(int dtype, const SegTables& t, OrderState* st, const GateRecord* rec, int nb, uint32_t tag,
                         int R, int nwrite, const uint64_t* local, bool keep_unused, Scale sc,
                         int blocks, bool nt, FlatBuckets flat, hipStream_t s) {
    if (blocks <= 0 || nb <= 0) return hipSuccess;
    const int keep = keep_unused ? 1 : 0;
    if (t.out != nullptr) {
        if (nwrite != 1 || flat.slab0 != nullptr) return hipErrorInvalidValue;
        switch (dtype) {
            case 1: return repair_dispatch<1, OUT_BINARY32>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
            case 2: return repair_dispatch<2, OUT_BINARY32>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
            default: return hipErrorInvalidValue;
        }
    }
    if (flat.slab0 != nullptr) {
        switch (dtype) {
            case 0: return repair_dispatch<0, OUT_FLAT>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
            case 1: return repair_dispatch<1, OUT_FLAT>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
            case 2: return repair_dispatch<2, OUT_FLAT>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
            default: return hipErrorInvalidValue;
        }
    }
    switch (dtype) {
        case 0: return repair_dispatch<0, OUT_GRAD>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
        case 1: return repair_dispatch<1, OUT_GRAD>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
        case 2: return repair_dispatch<2, OUT_GRAD>(nt, blocks, s, t, st, rec, nb, tag, R, nwrite, local, keep, sc, flat);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_probe(unsigned long long* word, unsigned long long value, long long wait_ticks,
                        hipStream_t waiter, hipStream_t writer) {
    hipLaunchKernelGGL(probe_wait_kernel, dim3(1), dim3(64), 0, waiter, word, value, wait_ticks);
    hipError_t e = after_launch();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(probe_write_kernel, dim3(1), dim3(64), 0, writer, word, value, wait_ticks);
    return after_launch();
}

hipError_t launch_pointer_copy(void** dst, void* const* src, int64_t count, unsigned* arrived, unsigned long long* done,
                               unsigned long long ticket, hipStream_t s) {
    if (count % 2 != 0) return hipErrorInvalidValue;
    const int64_t nvec = count / 2, round = 1024 * POINTER_COPY_LOADS;
    const int64_t blocks = std::min<int64_t>(std::max<int64_t>((nvec + round - 1) / round, 1), POINTER_COPY_BLOCKS);
    hipLaunchKernelGGL(blocks > 1 ? pointer_copy_kernel<true> : pointer_copy_kernel<false>, dim3(static_cast<unsigned>(blocks)), dim3(1024), 0, s,
                       reinterpret_cast<u32x4*>(dst), reinterpret_cast<const u32x4*>(src), nvec, static_cast<int>(blocks), arrived, done, ticket);
    return after_launch();
}

constexpr int64_t kStreamedGradients = int64_t(368) << 20;
bool accumulate_streams(int64_t ntiles, int R) { return ntiles * R * int64_t(TILE_BYTES) > kStreamedGradients; }

template <typename Micro>
static hipError_t accumulate_launch(const SegTables& t, int64_t ntiles, int R, const Micro& micro, unsigned lds, hipStream_t s) {
    if (ntiles <= 0 || R <= 0) return hipSuccess;
    dim3 grid(static_cast<unsigned>(ntiles), static_cast<unsigned>(R));
    // Up to about one and a half times the last-level cache (256 MiB) enough of the gradients is still
    // there for the next micro-step or the reduction to be worth plain accesses; beyond that the hint
    // pays.  R = 8, binary32, plain / with the hint, one micro-step: 183 MiB of gradients 91 / 96 us,
    // 290 MiB 145 / 149, 336 MiB 182 / 171, 397 MiB 219 / 202, 1 GiB (R = 32) 549 / 500; two micro-steps
    // and the reduction: 290 MiB 342 / 357, 336 MiB 406 / 411, 397 MiB 488 / 485.  ResNet-50 in bfloat16,
    // R = 8 (390 MiB): 207 / 198 us a micro-step; the first 37 BERT-large tensors, R = 32, four
    // micro-steps and the reduction: 15.0 / 13.8 ms.  A segment counts with whole tiles: lists of many
    // small tensors take the hint early and are no worse for it (two micro-steps and the reduction, real
    // bytes / whole tiles compared with the threshold: R = 64, 800 tensors of 500 bfloat16 404 / 390 us,
    // of 100 binary32 185 / 188; R = 32, 2000 of 500 bfloat16 442 / 429; R = 8, 8000 of 100 bfloat16 405 / 417).
    if (accumulate_streams(ntiles, R)) return launch(accumulate_kernel<true, Micro>, grid, lds, s, t, micro);
    return launch(accumulate_kernel<false, Micro>, grid, lds, s, t, micro);
}

hipError_t launch_accumulate(const SegTables& t, int64_t ntiles, int R, void* const* micro, unsigned lds, hipStream_t s) {
    return accumulate_launch(t, ntiles, R, MicroTable{micro}, lds, s);
}

template <int N>
static hipError_t accumulate_words(const SegTables& t, int64_t ntiles, int R, const uint64_t* words, int count, bool regular,
                                   unsigned lds, hipStream_t s) {
    MicroWords<N> m;
    std::memcpy(m.w, words, sizeof(uint64_t) * count);
    m.regular = regular ? 1 : 0;
    return accumulate_launch(t, ntiles, R, m, lds, s);
}

hipError_t launch_accumulate_by_value(const SegTables& t, int64_t ntiles, int R, const uint64_t* words, int count, bool regular,
                                      unsigned lds, hipStream_t s) {
    if (count > kMicroByValue) return hipErrorInvalidValue;
    if (count <= 64) return accumulate_words<64>(t, ntiles, R, words, count, regular, lds, s);
    if (count <= 192) return accumulate_words<192>(t, ntiles, R, words, count, regular, lds, s);
    return accumulate_words<kMicroByValue>(t, ntiles, R, words, count, regular, lds, s);
}

hipError_t launch_mask_write(uint64_t* dst, const uint64_t* masks, int count, const GateRecord* gate, uint32_t tag,
                             hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const dim3 grid((count + BLOCK - 1) / BLOCK);
    if (count > kMasksByValue) {
        hipLaunchKernelGGL(mask_write_kernel<MaskPointer>, grid, dim3(BLOCK), 0, s, dst, MaskPointer{masks}, count, gate, tag);
        return after_launch();
    }
    MaskPayload p;
    std::memcpy(p.m, masks, sizeof(uint64_t) * count);
    hipLaunchKernelGGL(mask_write_kernel<MaskPayload>, grid, dim3(BLOCK), 0, s, dst, p, count, gate, tag);
    return after_launch();
}

hipError_t launch_bitmap_or(uint64_t* local, uint8_t* global, uint64_t* host_global, uint64_t tag, const uint64_t* masks, int G, int R,
                            hipStream_t s) {
    if (G <= 0) return hipSuccess;
    const dim3 grid((G + BLOCK - 1) / BLOCK);
    if (masks_fit(R, G)) {
        MaskWords p;
        pack_masks(masks, G, R, p.m);
        p.first = 0;
        p.shift = mask_shift(R);
        hipLaunchKernelGGL(bitmap_or_kernel<MaskWords>, grid, dim3(BLOCK), 0, s, local, global, host_global, tag, p, G);
        return after_launch();
    }
    if (G > kMasksByValue) {
        hipLaunchKernelGGL(bitmap_or_kernel<MaskPointer>, grid, dim3(BLOCK), 0, s, local, global, host_global, tag, MaskPointer{masks}, G);
        return after_launch();
    }
    MaskPayload p;
    std::memcpy(p.m, masks, sizeof(uint64_t) * G);
    hipLaunchKernelGGL(bitmap_or_kernel<MaskPayload>, grid, dim3(BLOCK), 0, s, local, global, host_global, tag, p, G);
    return after_launch();
}

hipError_t launch_emit(int64_t ticks, void* const* ptrs, int R, int64_t nelem, int es,
                       int busy_blocks, float* sink, hipStream_t s) {
    // The delay and the copy are separate launches: a wait inside the copy's
    // blocks would start per block, and a grid with more blocks than fit on
    // the GPU at once would then wait several times the nominal delay.
    if (ticks > 0) {
        const unsigned bx = busy_blocks > 1 ? static_cast<unsigned>(busy_blocks) : 1u;
        hipLaunchKernelGGL(emit_kernel, dim3(bx, 1), dim3(BLOCK), 0, s, ticks,
                           static_cast<void* const*>(nullptr), R, int64_t(0), es,
                           busy_blocks > 0 ? 1 : 0, sink);
        const hipError_t e = after_launch();
        if (e != hipSuccess) return e;
    }
    if (ptrs == nullptr) return hipSuccess;
    int64_t want = (nelem + BLOCK * 8 - 1) / (BLOCK * 8);
    if (want < 1) want = 1;
    if (want > 1024) want = 1024;
    hipLaunchKernelGGL(emit_kernel, dim3(static_cast<unsigned>(want), static_cast<unsigned>(R)),
                       dim3(BLOCK), 0, s, int64_t(0), ptrs, R, nelem, es, 0, sink);
    return after_launch();
}

}  // namespace ddp
