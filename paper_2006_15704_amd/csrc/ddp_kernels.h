// Launch wrappers of the HIP kernels (gfx950).  Internal to the library.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace ddp {

// Work is cut into tiles of TILE_BYTES of gradient data: one thread block of
// BLOCK threads moves TILE_VECS 16-byte vectors per replica.  8 KiB tiles (two
// vectors per thread and replica) measured best: 16 KiB tiles with two or four
// vectors per thread were 1 to 4 points of HBM peak slower on the ResNet-50-
// and BERT-large-shaped lists under every cap on resident blocks.
constexpr int BLOCK = 256;
#ifndef DDP_TILE_VECS
#define DDP_TILE_VECS 512
#endif
constexpr int TILE_VECS = DDP_TILE_VECS;
constexpr int TILE_BYTES = TILE_VECS * 16;
constexpr int MAX_REPLICAS = 64;
// Short launches cut a tile into slices of one vector per lane of a wave.
constexpr int SLICE_BYTES = 1024;
constexpr int SLICES = TILE_BYTES / SLICE_BYTES;
// Threads that share the elements in vectors reaching over an end of a segment: at most 7 at each end.
constexpr int EDGE_SLOTS = 16;

// Dynamic LDS per block that leaves room for exactly `blocks` blocks on a compute unit with lds_per_cu bytes.  The hardware hands
// LDS out in units of 1280 bytes: an allocation between two of them takes the next one up.  (Rounded down to KiB
// instead, a third of 160 KiB left room for two blocks and a fifth for four.)
constexpr int64_t LDS_UNIT = 1280;
constexpr int64_t lds_for_blocks(int64_t lds_per_cu, int blocks) {
    return blocks <= 0 ? 0 : lds_per_cu / blocks / LDS_UNIT * LDS_UNIT;
}
constexpr bool lds_holds_exactly(int64_t lds_per_cu, int blocks) {
    const int64_t taken = (lds_for_blocks(lds_per_cu, blocks) + LDS_UNIT - 1) / LDS_UNIT * LDS_UNIT;
    return taken * blocks <= lds_per_cu && taken * (blocks + 1) > lds_per_cu;
}
// (eight blocks of four waves fill a unit's wave slots)
static_assert(lds_holds_exactly(160 * 1024, 1) && lds_holds_exactly(160 * 1024, 2) && lds_holds_exactly(160 * 1024, 3) &&
              lds_holds_exactly(160 * 1024, 4) && lds_holds_exactly(160 * 1024, 5) && lds_holds_exactly(160 * 1024, 6) &&
              lds_holds_exactly(160 * 1024, 7) && lds_holds_exactly(160 * 1024, 8), "a cap is the number of blocks it says");

// Launches of up to this many tiles take slices (es: bytes of an element).  Fused, the kernel alone, us, tile per block / slices,
// sixty tensors: binary32 R = 2, 128 tiles 4.0 / 4.1; R = 8, 128 4.8 / 4.6, 192 4.9 / 5.0, 256 6.0 / 6.8; R = 16, 128 6.7 / 6.6, 192 7.3 /
// 7.3, 256 9.1 / 9.8; R = 32, 128 10.7 / 9.8, 192 11.8 / 11.6 (two tensors 10.2 / 10.9); R = 64, 128 18.1 / 17.4, 192 20.4 / 22.4; bfloat16 R = 4,
// 192 5.1 / 4.9; R = 8, 192 5.9 / 5.3, 256 6.8 / 7.1; R = 16, 192 8.4 / 7.7, 256 10.8 / 10.5 (two tensors 9.2 / 9.6); R = 32, 192 13.2 / 12.9, 256
// 17.5 / 15.2 (15.0 / 16.0); R = 64, 128 21.2 / 19.1, 192 23.3 / 24.4.  Staged, us a synchronization: R = 4, 128 10.5 / 9.9, 256 11.5 / 11.5; R = 8,
// 256 14.6 / 13.9; R = 16, 256 22.7 / 21.0; R = 32, 256 42 / 36; R = 64, 128 50 / 37 (in two kernels, see split_pass in the host
// code, 36; 256 62 so, 67 in slices).
inline int64_t slice_tiles(int R, int es, bool staged) {
    if (R <= 4 || R > 32) return 128;
    return staged ? 256 : es == 2 ? 192 : 128;
}

// Slices that hold elements of a segment with `ntiles` tiles (whatever its lead-in).
inline int64_t slices_for(int64_t numel, int es, int64_t ntiles) {
    const int64_t most = ntiles * SLICES, n = (numel * es + 15 + SLICE_BYTES - 1) / SLICE_BYTES;
    return n < most ? n : most;
}

// Tiles up to which a launch takes slices where those that hold something are not listed (SegTables::slices): models above
// kListedSlices, and ddp_sync_static (a list is four bytes a slice; a context brings it to the device once, that call would on every
// call, and its 4 KiB of arguments do not hold it).  Blocks of empty slices end at once, but hold up others by the LDS they
// get.  GPU time of slices against tiles, %, by tiles of the launch; fused, binary32, 140 to 167 / 190 / 200 to 213 / 273:
// R = 9 to 16 -5 to -20 / -4 to -13 / -8 to +10 / +7 to +15, R = 17 to 24 -1 to -24 / +2 to -14 / +23 to -1 / +11, R = 32 +2 to -12 / - / +13 to +18 / +22;
// 16 bits, 200 to 234 / 250 to 262 / 320: R = 9 to 16 -5 to -22 / -3 to +10 / +13 to +18, R = 17 to 24 +11 to -7 / +1 to +4 / +8 to +11, R = 32 +7 to 0 / - / -.
// Staged, binary32, 261 to 322 / 339 to 385 / 427 / 480 to 547: R = 8 to 16 -11 to -16 / -6 to -14 / -3 to -6 / +3 to +17, R = 17 to 24 +6 to -4 / +1 to +9 / +9 to +11 / +9 to
// +16; bfloat16: R = 5 -2 to -12 / -8 to +8 / +14 / +24 to +34, R = 8 to 16 -12 to -21 / -4 to -18 / +2 to +6 / +9 to +26, R = 17 to 24 -2 to -8 / -6 to +2 / +2 to +3 / +2 to +6,
// R = 32 +2 to -2 / +2 / - / +19.
inline int64_t unlisted_tiles(int R, int es, bool staged) {
    if (staged) return R >= 8 && R <= 16 ? 384 : es == 2 && R >= 5 && R <= 24 ? 340 : 0;
    if (R < 9) return 0;
    return es == 2 ? (R <= 16 ? 240 : 0) : (R <= 24 ? 192 : 0);
}

// Whether a launch takes slices.  The tiles of small tensors are mostly empty.  Where the slices that hold something are listed
// they count, and the others have no block.  All marks in one call, 170 tensors of 200 kB in all / 240 of 600 / 240 of 1200, us, by tiles ->
// by listed slices: fused, binary32 R = 16 6.3 -> 5.3 / 6.8 -> 5.8 / -, R = 64 16.2 -> 7.1 / 19.9 -> 12.3 / -; bfloat16 R = 8 - / 6.1 -> 5.8 / 6.9 -> 5.8,
// R = 32 9.3 -> 5.6 / 12.2 -> 7.7 / 16.0 -> 11.2; staged, binary32 R = 8 - / 10.6 -> 9.2 / 13.6 -> 10.6, R = 32 13.9 -> 10.2 / 21.1 -> 14.8 / 27.1 -> 24.7;
// bfloat16 R = 16 10.7 -> 9.1 / 19.2 -> 11.8 / 24.8 -> 16.2, R = 64 27.3 -> 18.3 / 39.3 -> 30.3 / -.
inline bool takes_slices(int R, int es, bool staged, int64_t ntiles, int64_t nslices, bool listed) {
    const int64_t line = slice_tiles(R, es, staged);
    if (ntiles <= line) return true;
    return nslices <= line * SLICES && (listed || ntiles <= unlisted_tiles(R, es, staged));
}
// Whether a launch of slices goes by the list.  It is one more access in front of the others: 30 tensors of 300 kB, seven of ten slices of
// their tiles, R = 64 7.3 us without and 7.75 with it, R = 32 5.2 / 5.4.
inline bool takes_list(int R, int es, bool staged, int64_t ntiles, int64_t nslices) {
    return ntiles > slice_tiles(R, es, staged) || 2 * nslices < ntiles * SLICES;
}

// Tiles of a segment.  Vectors are cut at 16-byte boundaries of the
// destination, so a destination that starts `lead_bytes` (< 16) past such a
// boundary shifts the grid by that much; the caller passes the largest lead-in
// over all destinations the segment can have.
inline int64_t tiles_for(int64_t numel, int es, int lead_bytes) {
    if (numel <= 0) return 0;
    return (numel * es + lead_bytes + TILE_BYTES - 1) / TILE_BYTES;
}

// Device-resident tables over the G segments (parameters in bucket-major fill
// order) of the model.
struct SegInfo {               // 32 bytes, read with one scalar load
    int64_t numel;             // elements
    int64_t tile0;             // first tile of the segment in the global tile numbering
    int64_t flat_byte;         // byte offset of the segment inside a replica slab
    int32_t param;             // registration index
    int32_t flags;             // bits 0-7: element type; bit 8: all R gradient tensors share
                               // replica 0's address modulo 16; bits 16-19: that address
                               // modulo 16 (replica 0)
    __host__ __device__ int dtype() const { return flags & 0xFF; }
    __host__ __device__ bool congruent() const { return (flags & 0x100) != 0; }
    // bit 9 (binary32 outputs only): the output tensor's address modulo 16 equals twice
    // replica 0's address modulo 16, so whole input vectors map to whole output vectors
    __host__ __device__ bool out_congruent() const { return (flags & 0x200) != 0; }
    __host__ __device__ int lead_bytes() const { return (flags >> 16) & 0xF; }
};

struct SegTables {
    const SegInfo* seg;        // [G]
    const int32_t* tile_seg;   // [tiles] segment that each tile belongs to
    void* const* grad;         // [G*R + 16] replica r's gradient of segment g at [g*R+r]; sixteen
                               // null entries of padding so that any row can be read 16 wide
    void* const* out;          // [G] binary32 output tensor of segment g (lower-precision
                               // transport, Section 6.2.3), or null: averages go to the gradients
    int32_t G;
    int32_t R;
    const int32_t* slices = nullptr;   // [slices that hold elements] tile * SLICES + slice within it, in ascending order; null: there are
                                       // no such table, and slice launches have a block for every slice of their tiles
};

// The staged pipeline's flat buckets: replica r's slab at slab0 + r * stride (r < R), the averaged one
// at slab0 + R * stride; a segment lies flat_byte into each.  slab0 null = no flat buckets.
struct FlatBuckets {
    char* slab0;
    int64_t stride;
};

struct Scale {       // y = use_mul ? s * mul : s / div
    float div;
    float mul;
    int32_t use_mul;
};

// The division by R that turns the sum into DDP's average (Section 3.2.1).
inline Scale make_scale(int R) {
    Scale sc;
    sc.div = static_cast<float>(R);
    sc.mul = 1.0f / static_cast<float>(R);
    sc.use_mul = (R & (R - 1)) == 0;   // power of two: the reciprocal is exact, same bits as dividing
    return sc;
}

// All segment launches cover the tiles [tile_base, tile_base + ntiles) of the
// global tile numbering (tile0 / tile_seg).  `lds` in K2 and K4: bytes of
// dynamic LDS per block, beyond what the kernels use; they cap the number of
// blocks resident on a compute unit (0 = no cap).  The copy kernels K1 and K3
// keep one or two loads per thread in flight and want every block they can get.

// Timing: the next kernel launched on this thread through one of the pack / reduce / unpack /
// accumulate wrappers below carries `start` and `stop`; the runtime stamps them with the
// kernel's own start and end.  timing_pair_unused() clears the request and tells whether it
// was still pending (the wrapper had nothing to launch).
void time_next_launch(hipEvent_t start, hipEvent_t stop);
bool timing_pair_unused();

struct GateRecord;   // below, with the flag-ordering kernels

// gate (may be null): the record of the gate kernel enqueued in front of this
// launch; if gate->failed_tag == tag the launch does nothing.
// sig: where (null = nowhere) and with which ordinal the launch's last thread block reports that it
// has started (OrderState::dispatched)
struct DispatchSignal {
    unsigned long long* word;
    unsigned long long ord;
};

// K1: gradients -> flat replica slabs for all `nrep` replicas.  local (may be
// null = every replica used every parameter): one participation mask per
// segment; bit r = 0: write zeros into replica r's slot and do not read its tensor.
hipError_t launch_pack(const SegTables& t, int64_t tile_base, int64_t ntiles, char* slab0,
                       int64_t slab_stride, int nrep, const uint64_t* local,
                       const GateRecord* gate, uint32_t tag, hipStream_t s);

// K3: averaged slab -> gradient tensors of replicas [0, nrep).  global_used (may
// be null): per segment, 0 = no replica used the parameter; with keep_unused
// such parameters are not written.
hipError_t launch_unpack(const SegTables& t, int64_t tile_base, int64_t ntiles,
                         const char* out_slab, int nrep, const uint8_t* global_used, bool keep_unused,
                         hipStream_t s);

// K2 (staged): out[v] = scale(sum_r in_r[v]) over nvec 16-byte vectors;
// in_r = in0 + r*stride.
hipError_t launch_flat_reduce(int dtype, const char* in0, int64_t stride, char* out, int64_t nvec,
                              int R, Scale sc, bool nontemporal, unsigned lds,
                              const GateRecord* gate, uint32_t tag, DispatchSignal sig, hipStream_t s);

// Participation masks (bit r: replica r used the parameter) of the segments of a launch: none = every replica used every
// parameter; a table in device memory with one for every segment; or words that travel in the launch's arguments, a
// mask in the lowest 8, 16, 32 or 64 bits that hold R, those of segment `first` first.
constexpr int kMaskWords = 96;
struct Masks {
    const uint64_t* table = nullptr;
    const uint64_t* words = nullptr;
    int first = 0;
};
inline int mask_shift(int R) { return R <= 8 ? 3 : R <= 16 ? 4 : R <= 32 ? 5 : 6; }
inline bool masks_fit(int R, int64_t count) { return (count << mask_shift(R)) <= int64_t(kMaskWords) * 64; }
// words[0 .. kMaskWords) = masks[0 .. count), packed.
void pack_masks(const uint64_t* masks, int count, int R, uint64_t* words);

// K2 (fused): gather R replicas through the segment table, reduce, scatter to
// the gradient tensors of replicas [0, nwrite).  keep_unused as above
// (a replica with bit 0 contributes +0 and is not read; a parameter nobody
// used is skipped with keep_unused, else written as zeros).
// With flat.slab0 set (staged pipeline) the launch does K1's and K2's work in
// one pass instead: every replica's gradients are copied into its flat bucket
// (zeros for a replica that did not use the parameter) and the average goes to
// the averaged bucket; nwrite and keep_unused do not matter then.
// slice_base, nslices: the slices of the range that hold elements (slices_for), numbered through all segments.
hipError_t launch_fused_reduce(int dtype, const SegTables& t, int64_t tile_base, int64_t ntiles, int64_t slice_base, int64_t nslices,
                               int R, int nwrite, const Masks& masks, bool keep_unused, Scale sc,
                               bool nontemporal, unsigned lds, FlatBuckets flat,
                               const GateRecord* gate, uint32_t tag, DispatchSignal sig, hipStream_t s);
// (with t.out set -- 16-bit gradients, binary32 averages written to t.out -- nwrite must be 1)

// K2 (fused) without tables in device memory: they travel in the launch's arguments, as `count` words.
//   [0, n)           numel | congruent() << 31 | tile0 << 32 of every segment
//   then, as they are: the R pointers of every segment;
//   or, `regular`:     R bases and every segment's distance from them.
// (gradients of one type, all replicas take part, replica 0 receives the averages)
constexpr int kTableWords = 448;
struct WordTables {
    const uint64_t* words;
    int32_t n;
    bool regular;
    int64_t count(int R) const { return regular ? 2 * int64_t(n) + R : int64_t(n) * (R + 1); }
};
hipError_t launch_fused_reduce_by_value(int dtype, const WordTables& t, int64_t tile_base, int64_t ntiles, int64_t nslices, int R, Scale sc,
                                        hipStream_t s);

// ---- stream ordering through device flags -------------------------------------
// A bucket launch on a reduction stream must come after the backward-stream work
// that produces its gradients (Section 3.2.3).  Instead of an event pair per
// launch, the backward stream announces its position with a one-block kernel
// that stores a sequence number, and the reduction stream runs a one-wave gate
// kernel in front of the bucket kernel that polls for it.  The gate's wait is
// bounded; a gate that gives up marks its launch as failed, the bucket kernel
// that follows sees the mark and does nothing, and the repair launch enqueued by
// the finalizing step (when every gradient exists) redoes exactly those launches.
struct OrderState {
    unsigned long long ready_seq;   // latest announced sequence number (monotonic)
    unsigned long long pad0[15];    // the polled word has a cache line of its own
    uint32_t abort_tag;             // == iteration tag: a gate of this iteration has given up,
                                    //    later gates of the iteration give up at once
    uint32_t repaired;              // launches redone by repair launches since the context was created
    uint32_t pad1[30];
    unsigned long long dispatched;      // ordinal of the latest gated bucket launch whose last thread block
    unsigned long long pad2[15];        //    has started (monotonic): the launch is draining or done
};

struct GateRecord {                 // one per bucket, used by the launch whose first bucket it is
    int32_t tile_base;              // tile range of the launch
    int32_t ntiles;
    uint32_t failed_tag;            // == iteration tag: the gate gave up, the launch did nothing
    int32_t dtype;
};

// backward stream: ready_seq = seq.  (Everything enqueued before it on that stream has
// ended, and is visible device-wide, by the time the kernel that stores the number runs.)
// host (may be null): a word in pinned memory that receives the number as well, for the host to see.
hipError_t launch_announce(OrderState* st, unsigned long long seq, unsigned long long* host, hipStream_t s);

// backward stream, in front of a bucket launch that needs no gate there: the scheduling wait alone
hipError_t launch_chain_wait(OrderState* st, unsigned long long chain_ord, long long chain_ticks, hipStream_t s);

// The way back at the end of an iteration: on a reduction stream, behind its last bucket launch, *word = tag
// (host memory that a stream can wait on, hipStreamWaitValue64).
hipError_t launch_done(unsigned long long* word, unsigned long long tag, hipStream_t s);

// reduction stream: wait (at most wait_ticks of the device wall clock) until
// ready_seq >= need; on failure fill *rec, tag *row_summary (the record behind the last bucket's
// in the iteration's row: "a gate of this row gave up") and raise abort_tag.
// chain_ord / chain_ticks: once the number is there, the gate also waits (at most chain_ticks; 0 =
// not at all) until the bucket launch with ordinal chain_ord on ANOTHER reduction stream has
// started its last thread block, so that this launch fills the compute units as that one drains
// instead of sharing the memory system with it from its start.  A pure scheduling hint: the
// gate goes on when the bound is reached.
hipError_t launch_gate(OrderState* st, unsigned long long need, long long wait_ticks, GateRecord* rec,
                       GateRecord* row_summary, int32_t tile_base, int32_t ntiles, int32_t dtype, uint32_t tag,
                       unsigned long long chain_ord, long long chain_ticks, hipStream_t s);

// Redo the launches of element type `dtype` whose gate gave up in iteration `tag`
// (rec[0..nb)).  `blocks` persistent blocks; normally there is nothing to do.
hipError_t launch_repair(int dtype, const SegTables& t, OrderState* st, const GateRecord* rec, int nb, uint32_t tag,
                         int R, int nwrite, const uint64_t* local, bool keep_unused, Scale sc,
                         int blocks, bool nontemporal, FlatBuckets flat, hipStream_t s);

// Bounded probe (each wait at most wait_ticks): one wave on stream `waiter` stores `value` to word[2] and polls word[0] for it; one on stream
// `writer` waits for word[2] and then stores it to word[0].
// word[1] = 1 if the waiter saw the value, i.e. if the two streams run at the same time.  Streams that share a hardware
// queue run one after the other, and so does everything under tools that let one kernel run at a time: whichever of the
// two is first then waits in vain.
hipError_t launch_probe(unsigned long long* word, unsigned long long value, long long wait_ticks,
                        hipStream_t waiter, hipStream_t writer);

// Participation masks that travel in one launch's arguments (3 KiB); more are read from pinned memory.
constexpr int kMasksByValue = 384;

// dst[0 .. count) = masks: host memory, copied before the call returns; more than kMasksByValue: pinned
// memory that stays as it is until the launch has run.  gate / tag as for
// launch_fused_reduce: behind a gate that gave up nothing is written.
hipError_t launch_mask_write(uint64_t* dst, const uint64_t* masks, int count, const GateRecord* gate, uint32_t tag,
                             hipStream_t s);

// For g < G: local[g] = masks[g], global[g] = OR of its bits (the bitmap AllReduce of
// Section 4.2), host_global[g] = tag * 2 + the same bit.  masks as above, of R replicas; host_global: pinned.
hipError_t launch_bitmap_or(uint64_t* local, uint8_t* global, uint64_t* host_global, uint64_t tag, const uint64_t* masks, int G, int R,
                            hipStream_t s);

// dst[0 .. count) = src[0 .. count) (pinned memory; 16-byte aligned both, count even), then *done = ticket (pinned).
// arrived: a word in device memory that is 0 between launches; they run one after the other on one stream.
hipError_t launch_pointer_copy(void** dst, void* const* src, int64_t count, unsigned* arrived, unsigned long long* done,
                               unsigned long long ticket, hipStream_t s);

// Whether the gradients' loads and stores of a micro-step carry the non-temporal hint.
bool accumulate_streams(int64_t ntiles, int R);

// K4: grad[r][g] += micro gradient for all segments and replicas (null micro pointers are skipped).  ntiles = tile0[G].
// micro: a table in device memory, replica r's pointer of segment g at [g*R + r] (laid out as SegTables::grad, so that
// a block fetches both pointers at once) ...
hipError_t launch_accumulate(const SegTables& t, int64_t ntiles, int R, void* const* micro,
                             unsigned lds, hipStream_t s);

// ... or words that travel in the launch's arguments: the table itself, or with `regular` the addresses of R bases
// followed by the distances of the G segments from them (kMicroAbsent: a segment without a gradient).
constexpr int kMicroByValue = 448;
constexpr uint64_t kMicroAbsent = uint64_t(1) << 63;
hipError_t launch_accumulate_by_value(const SegTables& t, int64_t ntiles, int R, const uint64_t* words, int count, bool regular,
                                      unsigned lds, hipStream_t s);

// K6: a kernel that waits `ticks` of the device wall clock (bounded; skipped for
// ticks <= 0), followed by a kernel that copies src_r -> dst_r (nelem elements
// of es bytes) for r < R, where ptrs = [dst_0..dst_{R-1}, src_0..src_{R-1}] is a
// device array (null = delay only).  busy_blocks = 0: the delay is one block that
// sleeps between polls; > 0: that many blocks doing arithmetic between polls.
hipError_t launch_emit(int64_t ticks, void* const* ptrs, int R, int64_t nelem, int es,
                       int busy_blocks, float* sink, hipStream_t s);

}  // namespace ddp
