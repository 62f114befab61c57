// C ABI of the library: context, registration, bucket building, ready marks,
// finalize, no_sync accumulation and the synthetic backward emitter.  Host
// code only; the kernels are in ddp_kernels.hip.
#include "../../include/ddp_gfx950.h"

#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "bucket_plan.h"
#include "ddp_kernels.h"
#include "seg_layout.h"

namespace {

// Cross-stream ordering events: no timestamps, and a device-scope release --
// producer and consumer kernels run on the same GPU, so the default
// system-scope release (a cache write-back at every record) is not needed.
// Host-visible completion always goes through hipStreamSynchronize.
constexpr unsigned kOrderEvent = hipEventDisableTiming | hipEventReleaseToDevice;
// Timing events: device-scope release as well, so that the record itself does
// not add cache maintenance to the interval it measures.
constexpr unsigned kTimingEvent = hipEventReleaseToDevice;

thread_local std::string g_create_error;   // failures of calls that have no context

struct TimedLaunch {
    int32_t kind;
    int32_t bucket;
    hipEvent_t start, stop;
};

}  // namespace

struct ddp_ctx {
    int32_t R = 0;
    int32_t device = DDP_DEVICE_NONE;
    bool plan_only = true;
    hipStream_t reduce = nullptr, backward = nullptr;
    int64_t wall_clock_khz = 100000;

    // options
    int32_t pipeline = DDP_PIPELINE_STAGED;
    int32_t write_all = 0;
    int32_t timing = 0;
    int32_t nontemporal = 1;
    int64_t coalesce = -1;                        // > 0: consecutive buckets of one API call share a
                                                  // launch while it stays within this many bytes
    int32_t emit_busy_blocks = 0;                 // synthetic backward: 0 = sleeping delay kernel
    int32_t n_streams = -1;                       // reduction streams taken in turn by the launches; -1 = two
                                                  // for launches below cap_min_traffic, one for larger ones
    int32_t chain_launches = 1;                   // flag-ordered launches on alternating streams wait for their predecessor's last block
    unsigned long long launch_ord = 0;            // ordinal of the latest bucket launch that reports its dispatch (monotonic
                                                  // over the context's life)
    unsigned long long prev_launch_ord = 0;       // this iteration's latest such launch (0 = none yet), ...
    int prev_launch_lane = -1;                    // ... the reduction stream it went to (-1 = the backward stream) ...
    int64_t prev_launch_traffic = 0;              // ... the bytes it moves
    bool prev_launch_long = false;                // ... and whether it is a long one
    int32_t tail_on_backward = 1;                 // the call that completes an iteration launches on the backward stream
    int32_t blocks_per_cu = -1;                   // reduce kernels: resident blocks per compute unit (0 = no cap,
                                                  // -1 = chosen from R, see auto_blocks_per_cu)
    int64_t cap_min_traffic = int64_t(360) << 20; // ... applied to launches that move at least this many bytes
    bool cap_min_set = false;                     // ... by the caller's choice: shorter launches have no cap then
    int32_t acc_blocks_per_cu = -1;               // accumulate kernel: likewise, see auto_accumulate_blocks
    int64_t lds_per_cu = 160 * 1024;              // read from the device at creation

    bool registered = false, built = false;
    bool small_model = false;                     // set by build_internal, see kSmallModelTraffic
    bool wide = false;                            // some gradient is binary32
    ddp::BucketPlan plan;
    ddp::ReadyTracker tracker;
    std::vector<void*> grad_ptrs;            // [R][n], registration order
    std::vector<void*> out_ptrs;             // [n] binary32 output tensors (ddp_set_outputs), else empty

    // device memory owned by the library
    char* slabs = nullptr;                   // R input slabs followed by the output slab
    int64_t slab_stride = 0;
    std::vector<int64_t> bucket_slab_off;    // byte offset of each bucket inside a slab
    std::vector<int64_t> bucket_vecs;        // 16-byte vectors per bucket (padded)
    std::vector<int64_t> h_tile0, h_slices;  // [G+1], see HostTables
    void* d_tables = nullptr;                // one allocation holding all segment tables
    int32_t* d_tile_seg = nullptr;           // [tiles] segment index of every tile, and behind it the listed slices
    ddp::SegTables tables{};
    // participation: one mask per segment, bit r = replica r used the parameter
    int32_t find_unused = 0;                 // 1: parameters nobody used keep their gradients
    std::vector<uint64_t> local_cur;         // running iteration (entries of marked parameters are valid)
    std::vector<uint64_t> acc_used;          // recorded by ddp_no_sync_accumulate since the last finalize
    std::vector<uint64_t> micro_used;        // of the running ddp_no_sync_accumulate call
    std::vector<uint8_t> bucket_zero;        // per bucket: some bit of the running iteration is 0
    bool iter_zero = false;                  // any bit of the running iteration is 0
    int64_t iteration = 0;
    std::vector<uint8_t> global_closed;      // [n] host view of the closed iteration's global bitmap
    bool global_on_device = false;           // closed iteration: the bitmap kernel ran, result in h_global
    uint64_t* d_local = nullptr;             // [G]
    uint8_t* d_global = nullptr;             // [G]
    uint64_t* h_global = nullptr;            // [G], pinned, written by the bitmap kernel: iteration tag * 2 + bit; see await_bitmap
    uint64_t* h_masks[2] = {nullptr, nullptr};   // pinned copies of local_cur, by iteration parity; see stage_masks
    uint64_t masks_in_flight[2] = {0, 0};        // tag of the iteration whose kernels may still read h_masks, 0 = none
    int64_t masks_claimed_iter = -1;             // iteration for which h_masks was waited for
    void** d_micro = nullptr;                // [R * n, rounded up to an even number], and a word for pointer_copy_kernel
    // Pinned: micro_slots tables of micro-step pointers, used in turn, and behind them the ordinal of the latest
    // table that the device has read (written by pointer_copy_kernel).  Two keep the device busy: the host fills one while
    // the other has yet to be read (four micro-steps and the reduction, R = 2, four tensors, 37 us with one, 31.0 with
    // two, 31.6 with four; R = 32, 1600 tensors 1887 / 1876 / 1873; R = 64, 8000 tensors 19.5 ms with any).  Tables of at most
    // kSmallMicroTable bytes are four, so that the host of a short step is not held up by one that ran late.
    static constexpr size_t kSmallMicroTable = 64 * 1024;
    int micro_slots = 2;
    void** h_micro = nullptr;
    int64_t micro_table = 0;                 // pointers of one table
    unsigned long long micro_ticket = 0;     // ordinal of the latest call's table
    unsigned long long* micro_done() const { return reinterpret_cast<unsigned long long*>(h_micro + micro_slots * micro_table); }
    void** d_emit = nullptr;
    void** h_emit = nullptr;                 // pinned
    int64_t emit_cap = 0;                    // pointers
    std::vector<hipEvent_t> ev_ready;        // one per bucket
    hipEvent_t ev_done = nullptr, ev_emit = nullptr;
    bool emit_in_flight = false;

    std::vector<std::pair<int32_t, int32_t>> log_running, log_closed;
    std::vector<int32_t> order_running, order_closed;   // ready marks in the order they came (the trace)
    std::vector<uint8_t> used_running, used_closed;
    std::vector<TimedLaunch> timed;
    size_t open_group = static_cast<size_t>(-1);   // timing mode 2: the running iteration's entry
    // Reduction streams: lane 0 is the caller's reduce stream, lanes 1.. are created by the library
    // (DDP_OPT_REDUCE_STREAMS).  The launches of an iteration take the lanes in turn.
    static constexpr int kMaxLanes = 8;
    hipStream_t lane[kMaxLanes] = {};
    hipEvent_t ev_join[kMaxLanes] = {};           // lane's work of the iteration is done (event ordering)
    uint64_t* done_word[kMaxLanes] = {};          // likewise (flag ordering): the latest iteration tag whose launches on the lane have
                                                  // all ended, in memory that a stream can wait on
    hipEvent_t call_event = nullptr;              // backward-stream position of the running API call
    bool lane_used[kMaxLanes] = {};               // lane received work in the running iteration
    int latest_lane = 0;                          // lane of the latest launch on a reduction stream
    bool tail_chained = false;                    // the latest launch went to the backward stream, chained to one in front of it
    bool lane_ordered[kMaxLanes] = {};            // lane already waits for ev_call in the running API call
    int64_t launches_in_iter = 0;
    bool backward_idle_in_call = false;           // backward stream was found drained in this API call
    bool ordered_in_call = false;   // backward stream position of this API call already examined
    int32_t hold_marks = 0;         // DDP_OPT_LAUNCH_HOLD: a launchable bucket waits for up to this many
                                    // further ready marks for its successors to share its launch
    int32_t hold_until = 0;         // ready-mark count at which the held buckets go out at the latest
    std::vector<int32_t> deferred;  // buckets made launchable by the running API call, not yet enqueued

    // Stream ordering through device flags (DDP_OPT_FLAG_ORDER): the backward stream announces a
    // sequence number, a one-wave gate kernel in front of each bucket launch waits for it.
    int32_t flag_order = -1;                      // -1 = where the streams allow it, 0 = never (events)
    int64_t gate_wait_us = 100000;                // bound on one gate's wait
    int32_t num_cus = 256;                        // read from the device at creation
    char* d_order_mem = nullptr;                  // OrderState followed by the three probe words
    ddp::OrderState* d_order = nullptr;
    unsigned long long* d_probe = nullptr;
    // Gate records: kGateRows rows of one record per bucket plus one that summarizes the row
    // ("a gate of this iteration gave up"); iteration i uses row i % kGateRows.
    // Several iterations may be enqueued before the first one's repair launch has run, and a
    // gate of a later iteration that gives up early must not overwrite a record that an
    // earlier iteration's repair launch has yet to read.
    static constexpr int64_t kGateRows = 64;
    ddp::GateRecord* d_gate = nullptr;            // [kGateRows][buckets + 1], allocated with the buckets
    ddp::GateRecord* gate_row() const {
        return d_gate + (iteration % kGateRows) * (static_cast<int64_t>(plan.buckets.size()) + 1);
    }
    int64_t safe_iteration = 0;                   // everything enqueued before this iteration is known to be done
    uint64_t seq_issued = 0;                      // sequence numbers announced so far
    // Whether the GPU waits for the host (see kEarlyTraffic): the number of an announcement that is also
    // written to h_progress (pinned), 0 = none outstanding, and when it was enqueued; launches and bytes that may
    // still go to the backward stream on the strength of the last look; announcements of the running iteration that
    // came late, launches placed.
    unsigned long long* h_progress = nullptr;
    uint64_t progress_wait = 0;
    std::chrono::steady_clock::time_point progress_since;
    int32_t early_credit = 0, late_looks = 0, early_launches = 0;
    int64_t early_bytes = 0;
    int64_t early_total = 0;                      // launches placed since ddp_create
    uint64_t probe_value = 0;
    uint64_t call_seq = 0;                        // the number announced for the running API call
    bool call_by_flag = false;                    // the running API call orders its launches by flag
    bool lane_concurrent[kMaxLanes] = {};         // probed: the lane runs concurrently with the backward stream
    int64_t gates_in_iter = 0;                    // gate kernels enqueued in the running iteration
    std::string err;
};

namespace {

int32_t fail(ddp_ctx* c, int32_t code, const std::string& msg) {
    if (c) c->err = msg;
    else g_create_error = msg;
    return code;
}

#define HIPCHK(c, expr)                                                                    \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail((c), DDP_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

// Resident blocks per compute unit for long launches (lds_for_blocks turns them into LDS per block).
// A block keeps min(R, 8) x 2 loads per thread in flight, so with few
// replicas many blocks are needed.  The first 101 BERT-large tensors, all marks in one call, us with no cap (five blocks by
// registers) / four blocks / three / two: binary32 R = 3 271 / 265 / 276 / 309, R = 4 345 / 339 / 334 / 368, R = 5 430 / 423 / 414 /
// 442, R = 6 506 / 498 / 485 / 494, R = 8 663 / 652 / 634 / 623, R = 16 (60 tensors) 867 / 860 / 854 / 823; bfloat16 R = 3 132 / 132 / 138 / 163,
// R = 4 166 / 167 / 166 / 202, R = 8 327 / 327 / 320 / 315, R = 12 475 / 476 / 468 / 451, R = 16 624 / 624 / 620 / 596.
// (R = 2, no cap / four / two / one: binary32 215 / 218 / 252 / 326, bfloat16 99 / 99 / 141; R = 8 with one 685 and 399.)
// For R >= 16 one block is about as good on lists of large tensors but 6 points worse on the ResNet-50 list in
// fp16, whose many small tensors put slow boundary tiles on a unit that then
// has nothing else to run -- so two it is, also with binary32 outputs next to 16-bit
// inputs.
// copies: the staged pass, which writes as much as it reads (60 BERT-large tensors, us, no cap / three blocks / two: binary32 R = 2 332 /
// - / 338, R = 3 440 / - / 496, R = 4 551 / 540 / 540, R = 8 1002 / - / 1009; bfloat16 R = 2 170 / - / 181, R = 3 219 / - / 236, R = 4 278 / 272 /
// 264, R = 8 496 / - / 503).
// Three replicas are read by a round of two and one of one, so that a block has fewer loads under way than with four.
// write_all: every replica is written, too, and few replicas do best with few blocks (one launch of 900 MiB, us, no cap / four blocks / three /
// two: binary32 R = 2 201 / 197 / 199 / 216, R = 3 238 / 236 / 226 / 227, R = 4 263 / 266 / 262 / 247, R = 5 276 / 279 / 276 / 262, R = 8 300 / 302 /
// 305 / 306, R = 12 319 / 319 / 319 / 325, R = 16 330 / 329 / 328 / 337; bfloat16 R = 2 199 / 199 / 201 / 235, R = 3 241 / 241 / 228 / 233, R = 4 261 /
// 260 / 259 / 251, R = 5 278 / 278 / 281 / 264, R = 8 296 / 296 / 299 / 295, R = 12 321 / 321 / 325 / 324, R = 16 331 / 331 / 332 / 338; sixty
// BERT-large tensors, binary32 R = 4 412 / 418 / 412 / 385, R = 8 849 / 852 / 835 / 851, R = 10 1067 / 1093 / 1063 / 1049, R = 12 1301 / 1314 / 1307 / 1294,
// R = 16 1756 / 1760 / 1748 / 1748, R = 32 3623 / 3627 / 3609 / 3528; bfloat16 R = 8 420 / 421 / 426 / 415, R = 10 530 / 530 / 535 / 524, R = 12 647 / 647 / 656 /
// 647, R = 14 755 / 755 / 762 / 766, R = 16 870 / 871 / 876 / 886, R = 32 1812 / 1810 / 1807 / 1786).
// Three blocks, lists of 2.2 GB moved, all marks in one call, us with four blocks / three / two: binary32 R = 4 344 / 341 / 379, R = 5 348 / 340 / 367, R = 6
// 353 / 341 / 347, R = 7 359 / 348 / 352, R = 8 368 / 354 / 340; bfloat16 R = 4 342 / 346 / 426, R = 5 351 / 342 / 390, R = 6 360 / 347 / 364, R = 7 367 / 353 /
// 373, R = 8 378 / 370 / 345; binary16 R = 4 346 / 342 / 399 (120 MiB buckets, one mark per call 355 / 359 / 403), R = 5 355 / 342 / 393, R = 6 358 / 346 / 378, R = 7
// 370 / 354 / 367, R = 8 377 / 363 / 354; binary32 averages R = 4 412 / 428 / 455, R = 5 418 / 415 / 441, R = 6 418 / 414 / 420, R = 7 414 / 413 / 395; every
// replica written, no cap / three / two: binary32 R = 3 573 / 543 / 544, R = 16 774 / 771 / 796, bfloat16 R = 3 570 / 550 / 579, R = 16 772 / 777 / 791.  Sixty BERT-large
// tensors, three / two: binary32 R = 6 325 / 328, R = 7 376 / 373, every replica written R = 3 294 / 282; bfloat16 R = 6 164 / 171, R = 7 189 / 196, every replica
// written R = 3 145 / 148.
int32_t auto_blocks_per_cu(int32_t R, int es, bool copies, bool write_all, bool out32) {
    if (copies) return R == 4 ? 2 : 0;
    if (write_all) return R <= 2 || (R >= 12 && R <= 16) ? 0 : R == 3 && es == 2 ? 3 : 2;
    if (R <= 2) return 0;
    if (R == 3 || (R == 4 && es == 2)) return 4;
    return R <= (out32 || es == 4 ? 6 : 7) ? 3 : 2;
}

// Resident blocks of the accumulation.  Gradients that go past the caches: four, in 16 bits three; others have less of the memory to wait for
// and are over sooner, so that more blocks under way count for more.  Us a micro-step of 60 tensors, three / four / five / six / no cap:
// 2.4 GB of gradients, binary32 R = 2 1169 / 1144 / 1162 / 1183 / 1204, R = 32 1169 / 1170 / 1194 / 1211 / 1243; bfloat16 R = 2 1135 / 1152 / 1168 / 1186 / 1192, R = 8
// 1132 / 1165 / 1181 / 1204 / 1218; binary16 R = 8 1152 / 1173 / 1185 / 1205 / 1223; 800 MB, binary32 R = 8 394 / 382 / 383 / 392 / 399, bfloat16 370 / 377 / 387 / 392 / 394; 200
// MB, binary32 R = 2 108 / 103 / 102 / 100 / 101, R = 8 106 / 104 / 104 / 103 / 103, bfloat16 R = 8 101 / 102 / 101 / 102 / 103; 60 MB, binary32 R = 2 34.1 / 33.3 / 32.1 / 30.0 /
// 29.7, R = 8 34.3 / 32.5 / 31.2 / 30.1 / 29.7, bfloat16 R = 8 31.7 / 30.3 / 30.1 / 29.9 / 29.8.
int32_t auto_accumulate_blocks(bool streamed, bool wide) { return streamed ? (wide ? 4 : 3) : (wide ? 6 : 5); }

// Bytes of bucket data up to which buckets that become launchable together share a launch: a launch pays its start-up and drain, and
// very long ones lose a little throughput again.  Lists of 5 to 6 GB in all, us, limits of MiB: R = 2 binary32 400 941, 800
// 933, 1600 941, bfloat16 969, 957, 961; R = 3 240 463, 480 452; R = 4 240 974, 480 970, 960 975, bfloat16 960, 959, 973, binary16 986, 990, 996; R = 5
// 100 645, 200 636, 400 640; R = 6 100 666, 200 644; R = 8 100 960, 200 948, 400 950, 800 961, bfloat16 986, 966, 961; R = 16 70 980, 140 972, 280 973; R = 24, 4 GB, 50
// 653, 100 657; R = 32 50 965, 100 960; R = 64 50 805, 100 808; BERT-large, R = 8 100 1958, 200 1934, 400 1935, 800 1946.
// Launches that write more do not gain from twice the bytes: every replica written, R = 4 240 775, 480 778; staged, R = 8 100 1148, 200 1155,
// R = 16 70 1160, 140 1172; binary32 averages, R = 8 100 711, 200 712, R = 16 70 724, 140 731.
int64_t auto_coalesce(int32_t R) {
    const int64_t mib = int64_t(1) << 20;
    return (R <= 2 ? 400 : R <= 4 ? 240 : R <= 8 ? 100 : R <= 16 ? 70 : 50) * mib;
}

// What a launch hold fills a launch with, and 0 = no sharing.
int64_t coalesce_limit(const ddp_ctx* c) { return c->coalesce < 0 ? auto_coalesce(c->R) : c->coalesce; }

int64_t launch_limit(const ddp_ctx* c) {
    const bool one_writer = c->pipeline == DDP_PIPELINE_FUSED && !c->write_all && c->out_ptrs.empty();
    const bool twice = c->coalesce < 0 && one_writer && c->R != 4 && c->R <= 16;
    return coalesce_limit(c) * (twice ? 2 : 1);
}

// What is left of a run of buckets goes out with its last launch if it is at most a quarter of the limit that the library chose: a
// launch of its own would be mostly start-up and drain, on another stream and with the way back from it.  One launch of 1.1 /
// 1.25 / 1.5 times the limit (of the former limits for one writer) against two, %: binary32 R = 2 -3.9 / -2.0 / -1.2, R = 4 -2.8 / -1.4 / -0.6, R = 8 -4.9 /
// -3.1 / -2.3, R = 16 -2.9 / -1.8 / -0.8, R = 32 -1.8 / -0.7 / +0.3; binary32 averages R = 2 -3.1 / -1.8 / +0.3, R = 8 -4.9 / -5.2 / -2.2, R = 32 -1.8 / -0.9 / +0.1;
// staged R = 2 -1.7 / -0.7 / +0.4 (bfloat16 -1.1 / +0.6 / +2.5), R = 4 -2.2 / -1.1 / -0.8, R = 8 -1.6 / -0.2 / +0.6, R = 16 -1.3 / -0.1 / +0.4; every
// replica written R = 4 -2.4 / -2.3 / -0.3, R = 8 -1.8 / -1.5 / +0.7, R = 16 -1.4 / -1.0 / -0.1.  The ragged list, R = 8, 114 MiB, 188.5 / 179.5 us.
int64_t last_launch_limit(const ddp_ctx* c) {
    const int64_t limit = launch_limit(c);
    return c->coalesce < 0 ? limit + limit / 4 : limit;
}

// A launch is chained to the one in front of it if that one moves at least this many bytes.
constexpr int64_t kChainMinTraffic = int64_t(160) << 20;

// Whether a launch's kernels carry the gate check and report the dispatch: always but for the staged
// pipeline with its kernels timed one by one.
bool carries_gate(const ddp_ctx* c) { return c->pipeline == DDP_PIPELINE_FUSED || c->timing != 1; }

// Bytes that a launch over `launch_bytes` of bucket data moves (the staged pass writes R copies too).
int64_t launch_traffic(const ddp_ctx* c, int64_t launch_bytes) {
    return launch_bytes * (c->pipeline == DDP_PIPELINE_FUSED ? c->R + 1 : 2 * c->R + 1);
}

// Staged: whether a launch copies and reduces in two kernels.  The one pass over tiles sums
// a tile's replicas in one block, chunk after chunk; with many replicas and few tiles most of the chip
// idles meanwhile, where the copies run in a block per tile and replica.  (Still fewer tiles go in slices.)
// One pass / two kernels, us a synchronization, all marks in one call, sixty tensors: binary32, 384 tiles R = 24 40 / 40,
// R = 32 53 / 49, R = 64 102 / 87, 512 R = 64 147 / 122; 16 bits, 384 R = 24 48 / 45, R = 64 118 / 97, 512 R = 24 56 / 52,
// R = 32 74 / 64, R = 64 149 / 117, 1024 R = 32 143 / 144.  R = 16 in one pass is no slower.
bool split_pass(const ddp_ctx* c, int32_t dtype, int64_t ntiles, int64_t nslices) {
    if (c->nontemporal != 0 && ddp::takes_slices(c->R, ddp::elem_size(dtype), true, ntiles, nslices, c->tables.slices != nullptr)) return false;
    return c->R > 16 && ntiles <= (dtype == DDP_FP32 ? 512 : 1024);
}

// A model of at most kSmallModelBuckets buckets that move less than this together keeps all of its
// launches on the backward stream, unless the caller asked for a number of reduction streams or for
// launches that all go to them (DDP_OPT_TAIL_ON_BACKWARD 0).  Such a
// launch takes 3 to 4 us there; to have it on a reduction stream the backward stream runs an
// announcement of 1.5 us and the host makes three launches instead of one (2.3 us each), and the way
// back costs two to four of each and an event pair per stream.  Eight small tensors in three buckets,
// R = 2, one mark per call, staged: 70 us a synchronization with reduction streams, 13 us without.
// Under a running backward pass every launch but the last exposes all of its own time, which grows
// with R (a block sums its replicas one chunk after the other), instead of its announcement.  Twelve
// tensors, 40 us of backward work each, exposed time with reduction streams / without, fused, 0.1 to
// 3.5 MiB moved: R = 2 and 4, four buckets, 19 to 25 / 12 to 20 us; R = 8, three buckets 21 to 25 /
// 17 to 22, four 25 to 27 / 24 to 30; R = 16, two buckets 16 to 21 / 8 to 19, four 25 to 28 / 18 to 38;
// R = 32, two 18 to 32 / 12 to 42, four 24 to 41 / 26 to 86; R = 64, four 28 to 37 / 39 to 78.  So the
// line is R x (buckets - 1) <= kSmallModelReplicas.  (ResNet-50 in 161 buckets, R = 16: 0.29 / 0.81 ms.)
constexpr int64_t kSmallModelTraffic = int64_t(4) << 20;
constexpr int32_t kSmallModelBuckets = 4;
constexpr int64_t kSmallModelReplicas = 16;

// Whether a launch over `launch_bytes` of bucket data is a long one: the cap on resident
// blocks pays, and a second reduction stream does not, from about 360 MiB of traffic on
// (R = 8: 40 MiB of bucket data; R = 32: every 25 MiB bucket, 72.0 against 69.4 % of peak with
// one mark per call; R = 16 likewise 71.7 against 69.4 %).
// The count is (R + 1) x bucket bytes in both pipelines, for the streams that launches take in turn, for
// the cap and for whether two neighbours on two streams are chained.  Staged, one mark per
// call, 25 MiB buckets: BERT-large, R = 8, 4.73 ms when neighbours counted as long by the bytes they
// move and as short so took two streams unchained, 4.67 chained on two streams, 4.82 on one stream.
bool long_launch(const ddp_ctx* c, int64_t launch_bytes) {
    return launch_bytes * (c->R + 1) >= c->cap_min_traffic;
}

unsigned lds_for_blocks(const ddp_ctx* c, int32_t blocks) {
    return static_cast<unsigned>(ddp::lds_for_blocks(c->lds_per_cu, blocks));
}

// Resident blocks of shorter launches (which take tiles): one mark per call, us, no cap / four blocks / two: BERT-large, R = 8,
// 2034 / 2025 / 2038, 240 MB in 8 MiB buckets, R = 12, 555 / 553 / 555, ResNet-50-sized, binary16, R = 16 369 /
// 366 / 357; 120 MB, R = 4 230 / 230 / 249; all marks in one call, 16 MB, R = 8 25.1 / 25.0 / 25.5 (bfloat16 25.4 / 25.5 / 26.7), R = 16 46.5 / 46.5 /
// 45.7.
// Three for binary32 launches that move 200 MiB and more and write the averages once.  Ten buckets, % of the time with four, launches of 205 / 225 /
// 250 / 300 / 350 MiB: R = 8 +0.5 / -0.4 / -1.4 / -2.2 / -1.4, R = 9 -1.2 / -1.1 / -0.5 / -1.5 / -2.1, R = 10 -0.3 / -1.6 / -3.1 / -3.5 / -2.0, R = 12 -2.2 / -1.5 / -2.4 /
// -1.9 / -2.1, R = 15 -1.8 / -1.4 / -1.5 / -2.4 / -1.5; BERT-large in 25 MiB buckets R = 8 -2.3, R = 10 -1.9, R = 12 -0.3 (runs of one side differ by 0.5 to
// 1.5).  Below, R = 8 in 72 MiB launches +1.3.  Every replica written it gains nothing: R = 8 -0.4 / -0.5 / -0.6 / +0.3 / -0.1 and BERT-large +1.2, R = 12 +0.7 / +0.3 /
// +0.4 / +0.1 / -0.5, R = 14 +0.6 / +0.3 / +0.6 / 0 / +0.5.  Nor do (us, three / four blocks) bfloat16, R = 10 205.2 / 203.8, binary32 averages, R = 8 404 / 402, masks,
// ResNet-50, R = 8 127.4 / 124.4, R = 5, 240 MiB 204.4 / 202.1; R = 16, 212 MiB 207.9 with three and 205.0 with two.
constexpr int64_t kThreeBlocksFrom = int64_t(200) << 20;
int32_t short_launch_blocks(int32_t R, int64_t moved, int es, bool masked, bool write_all) {
    if (R <= 4) return 0;
    if (R >= 16) return 2;
    return R >= 8 && es == 4 && moved >= kThreeBlocksFrom && !masked && !write_all ? 3 : 4;
}

unsigned occupancy_lds(const ddp_ctx* c, int64_t launch_bytes, int es, bool copies, bool masked) {
    if (c->blocks_per_cu >= 0) return long_launch(c, launch_bytes) ? lds_for_blocks(c, c->blocks_per_cu) : 0;
    if (long_launch(c, launch_bytes)) return lds_for_blocks(c, auto_blocks_per_cu(c->R, es, copies, c->write_all, !c->out_ptrs.empty()));
    return copies || c->cap_min_set ? 0 : lds_for_blocks(c, short_launch_blocks(c->R, launch_bytes * (c->R + 1), es, masked, c->write_all));
}

using ddp::make_scale;

// DDP_OPT_TIMING = 1: the launch between timed_begin and timed_end (exactly one kernel) carries a
// pair of events stamped with the kernel's own start and end.
int32_t timed_begin(ddp_ctx* c, int32_t kind, int32_t bucket, hipStream_t s, size_t* slot) {
    (void)s;
    *slot = static_cast<size_t>(-1);
    if (c->timing != 1) return DDP_OK;
    TimedLaunch t{kind, bucket, nullptr, nullptr};
    HIPCHK(c, hipEventCreateWithFlags(&t.start, kTimingEvent));
    HIPCHK(c, hipEventCreateWithFlags(&t.stop, kTimingEvent));
    ddp::time_next_launch(t.start, t.stop);
    c->timed.push_back(t);
    *slot = c->timed.size() - 1;
    return DDP_OK;
}

int32_t timed_end(ddp_ctx* c, size_t slot, hipStream_t s) {
    if (slot == static_cast<size_t>(-1)) return DDP_OK;
    if (ddp::timing_pair_unused()) {
        // nothing was launched (an empty range): an empty interval on the stream
        HIPCHK(c, hipEventRecord(c->timed[slot].start, s));
        HIPCHK(c, hipEventRecord(c->timed[slot].stop, s));
    }
    return DDP_OK;
}

void drop_timed(ddp_ctx* c) {
    for (TimedLaunch& t : c->timed) {
        if (t.start) (void)hipEventDestroy(t.start);
        if (t.stop) (void)hipEventDestroy(t.stop);
    }
    c->timed.clear();
    c->open_group = static_cast<size_t>(-1);
}

void look_at_progress(ddp_ctx* c);

// A new API call begins: whatever the caller enqueued on the backward stream
// since the last call has to be ordered before the launches of this one.
void new_call(ddp_ctx* c) {
    if (c->progress_wait != 0) look_at_progress(c);
    c->call_by_flag = false;
    c->ordered_in_call = false;
    c->backward_idle_in_call = false;
    c->call_event = nullptr;
    for (bool& b : c->lane_ordered) b = false;
}

// Whether stream `waiter` makes progress while stream `other` is busy and vice versa.  HIP
// streams that share a hardware queue run one after the other.  The probe is a bounded wait on
// `waiter` for a value written from `other`, which waits for the waiter first: streams that passed it run at the same
// time, as the gates need, and the value waits at the end of an iteration, which the runtime makes with a kernel that polls
// as long as it takes: under a tool that lets one kernel run at a time both would be in each other's way, and events are used.
int32_t probe_pair(ddp_ctx* c, hipStream_t waiter, hipStream_t other, bool* concurrent) {
    *concurrent = false;
    if (waiter == other) return DDP_OK;
    HIPCHK(c, hipStreamSynchronize(waiter));
    HIPCHK(c, hipStreamSynchronize(other));
    ++c->probe_value;
    HIPCHK(c, ddp::launch_probe(c->d_probe, c->probe_value, 300 * c->wall_clock_khz / 1000, waiter, other));
    HIPCHK(c, hipStreamSynchronize(waiter));
    HIPCHK(c, hipStreamSynchronize(other));
    unsigned long long seen = 0;
    HIPCHK(c, hipMemcpy(&seen, c->d_probe + 1, sizeof(seen), hipMemcpyDeviceToHost));
    *concurrent = seen == 1;
    return DDP_OK;
}

// Words that streams wait on (hipMallocSignalMemory gives them out one at a time, and an allocation takes 30 us): contexts hand
// theirs on, by device, when their streams have ended; at most kSpareWords are kept.
constexpr size_t kSpareWords = 32;
std::mutex g_words_mu;
std::vector<std::pair<int, uint64_t*>> g_spare_words;

uint64_t* take_word(int device) {
    {
        std::lock_guard<std::mutex> lock(g_words_mu);
        for (size_t k = g_spare_words.size(); k-- > 0;)
            if (g_spare_words[k].first == device) {
                uint64_t* const w = g_spare_words[k].second;
                g_spare_words.erase(g_spare_words.begin() + static_cast<std::ptrdiff_t>(k));
                __atomic_store_n(w, uint64_t(0), __ATOMIC_SEQ_CST);
                return w;
            }
    }
    int can = 0;
    void* p = nullptr;
    hipPointerAttribute_t at{};
    if (hipDeviceGetAttribute(&can, hipDeviceAttributeCanUseStreamWaitValue, device) != hipSuccess || can == 0 ||
        hipExtMallocWithFlags(&p, sizeof(uint64_t), hipMallocSignalMemory) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeHost) {      // (the host sets them to 0)
        (void)hipGetLastError();
        (void)hipFree(p);
        return nullptr;
    }
    __atomic_store_n(static_cast<uint64_t*>(p), uint64_t(0), __ATOMIC_SEQ_CST);
    return static_cast<uint64_t*>(p);
}

// No stream waits for the word or writes it any more.
void give_word(int device, uint64_t* w) {
    {
        std::lock_guard<std::mutex> lock(g_words_mu);
        if (g_spare_words.size() < kSpareWords) {
            g_spare_words.emplace_back(device, w);
            return;
        }
    }
    (void)hipFree(w);
}

// The word that the backward stream waits on for lane l (0 at first).  A device that cannot have one keeps events.
bool make_done_word(ddp_ctx* c, int l) {
    if (c->done_word[l] == nullptr) c->done_word[l] = take_word(c->device);
    return c->done_word[l] != nullptr;
}

// Lane l against the backward stream: a gate kernel on a lane that shares the backward
// stream's hardware queue would keep the announcement it waits for from running, so such
// pairs keep events.
int32_t probe_lane(ddp_ctx* c, int l) {
    const int32_t rc = probe_pair(c, c->lane[l], c->backward, &c->lane_concurrent[l]);
    if (rc == DDP_OK && c->lane_concurrent[l]) c->lane_concurrent[l] = make_done_word(c, l);
    return rc;
}

// Creates reduction stream l (default priority, no implicit ordering with the legacy
// default stream).  A new stream may land on the hardware queue of the backward stream, or
// on that of the caller's reduction stream, next to which it is meant to run; a few more are
// tried then (the misfits are destroyed once one fits, so that the next try does not get the
// same queue again).  A stream that runs side by side with both is taken at once; failing
// that, the first one that does so with the backward stream.
int32_t create_lane(ddp_ctx* c, int l) {
    if (c->lane[l]) return DDP_OK;
    hipStream_t tried[7];
    int n_tried = 0, second_best = -1, best = -1;
    while (n_tried < 7 && best < 0) {
        hipStream_t s = nullptr;
        HIPCHK(c, hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
        tried[n_tried] = s;
        bool with_backward = false, with_first = true;
        int32_t rc = probe_pair(c, s, c->backward, &with_backward);
        if (rc == DDP_OK && with_backward && c->lane[0] != c->backward) rc = probe_pair(c, s, c->lane[0], &with_first);
        if (rc != DDP_OK) {
            for (int k = 0; k <= n_tried; ++k) (void)hipStreamDestroy(tried[k]);
            return rc;
        }
        if (with_backward && with_first) best = n_tried;
        else if (with_backward && second_best < 0) second_best = n_tried;
        ++n_tried;
    }
    const int pick = best >= 0 ? best : second_best >= 0 ? second_best : n_tried - 1;
    c->lane[l] = tried[pick];
    c->lane_concurrent[l] = (best >= 0 || second_best >= 0) && make_done_word(c, l);
    for (int k = 0; k < n_tried; ++k)
        if (k != pick) (void)hipStreamDestroy(tried[k]);
    HIPCHK(c, hipEventCreateWithFlags(&c->ev_join[l], kOrderEvent));
    return DDP_OK;
}

// Flags order the launches of the running API call if every reduction stream in use passed
// the probe.
bool flags_usable(const ddp_ctx* c) {
    if (c->flag_order == 0 || !carries_gate(c) || c->d_gate == nullptr) return false;
    // (by default the second stream is only used if it passed the probe, see launch_range)
    const int lanes = c->n_streams < 0 ? 1 : c->n_streams;
    for (int l = 0; l < lanes; ++l)
        if (!c->lane_concurrent[l]) return false;
    return true;
}

// A short launch on a reduction stream costs the host three launches (announcement, gate, kernel, 3 us each), on the
// backward stream one, but there it holds the backward pass up for its own time.  That does not matter while the GPU
// waits for the host anyway.  So the announcement of a short launch is shown to the host as well, and if it shows
// within kPromptUs, which takes a backward stream with nothing left to run, the next short launches of the iteration go to
// the backward stream, kEarlyLaunches of them that move kEarlyBytes (50 us of the GPU) at most; then one is announced again.  A
// stream that is busy with the backward pass does not get there in time, and after kLateLooks announcements (and one for
// every four launches placed) that came late no more are shown.
// One mark per call, us a synchronization, without / with (several processes, whose launches take the host more or less time): ResNet-50
// in 1 MiB buckets, binary16, R = 16, 404 to 503 / 283 to 343; 19 MB in 62 buckets, binary32, R = 24, 470 to 589 / 317 to 319; 40 MB in 13,
// bfloat16, R = 4, 100 to 135 / 86 to 94; 23 MB in 5, R = 8, 89 to 115 / 78 to 85; every replica written, 17 MB in 12, R = 8, 187 to 193 / 116
// to 123; 90 buckets of 900 elements with participation masks, R = 8, 1090 to 1500 / 670 to 880.  Exposed under 10 us of backward work a parameter,
// ResNet-50 in 1 MiB buckets, fused 96 to 122 / 94 to 134, staged 152 to 163 / 143 to 164 (with the bucket's mark in place of kPromptUs,
// which lets the GPU be up to a bucket behind, 125 / 182 and 155 / 235).
constexpr int64_t kEarlyTraffic = int64_t(64) << 20, kEarlyBytes = int64_t(256) << 20;
constexpr int32_t kEarlyLaunches = 16, kLateLooks = 3, kPromptUs = 8;

// The host looks behind every launch of its own.  A number that is there within kPromptUs came in time, one
// that is not there after kPromptUs comes late; one that is there by then but was last looked for before says
// nothing of the stream, only that the host took long, and counts as neither.
void look_at_progress(ddp_ctx* c) {
    if (c->progress_wait == 0) return;
    // (the clock first: what is not there yet a little later was not there then)
    const bool late = std::chrono::steady_clock::now() - c->progress_since > std::chrono::microseconds(kPromptUs);
    const bool reached = __atomic_load_n(c->h_progress, __ATOMIC_RELAXED) >= c->progress_wait;
    if (!reached && !late) return;
    c->progress_wait = 0;
    if (!reached) {
        ++c->late_looks;
    } else if (!late) {
        c->early_credit = kEarlyLaunches;
        c->early_bytes = kEarlyBytes;
    }
}

// Whether the launch at hand goes to the backward stream on the strength of the last look.
bool take_early(ddp_ctx* c, int64_t traffic) {
    look_at_progress(c);
    if (c->early_credit != 0 && traffic > c->early_bytes) c->early_credit = 0;
    if (c->early_credit == 0) return false;
    c->early_bytes -= traffic;
    --c->early_credit;
    ++c->early_launches;
    ++c->early_total;
    return true;
}

// Order the launches of the running API call after the gradient-producing work enqueued so
// far: one look at the backward stream, and at most one announcement or event on it, serves
// every bucket the call launches (the caller cannot enqueue anything in the middle of a call).
// If the backward stream has already drained there is nothing to wait for.
// look: the host will want to know when the stream gets there.
int32_t order_call(ddp_ctx* c, int32_t first, bool look) {
    if (c->ordered_in_call) return DDP_OK;
    // (a stream that is being captured into a graph cannot be queried: treat it as busy)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool capturing = hipStreamIsCapturing(c->backward, &cap) == hipSuccess &&
                           cap != hipStreamCaptureStatusNone;
    const bool by_flag = !capturing && flags_usable(c);
    // With flags the announcement is enqueued without first asking whether the backward
    // stream has drained: the question (a stream query takes as long on the host as
    // two launches) would only save the two small kernels when it has.
    const hipError_t q = (capturing || by_flag) ? hipErrorNotReady : hipStreamQuery(c->backward);
    if (q == hipErrorNotReady) {
        if (by_flag) {
            // a one-block kernel instead of an event record (which stalls the stream
            // for about 12 us here)
            c->call_seq = ++c->seq_issued;
            const bool show = look && c->late_looks < kLateLooks + c->early_launches / 4;
            HIPCHK(c, ddp::launch_announce(c->d_order, c->call_seq, show ? c->h_progress : nullptr, c->backward));
            if (show) {
                c->progress_wait = c->call_seq;
                c->progress_since = std::chrono::steady_clock::now();
            }
            c->call_by_flag = true;
        } else {
            HIPCHK(c, hipEventRecord(c->ev_ready[first], c->backward));
            c->call_event = c->ev_ready[first];
        }
    } else if (q == hipSuccess) {
        c->backward_idle_in_call = true;
        c->safe_iteration = c->iteration;     // every earlier iteration has finished
    } else {
        return fail(c, DDP_ERR_HIP, std::string("hipStreamQuery: ") + hipGetErrorString(q));
    }
    c->ordered_in_call = true;
    return DDP_OK;
}

// Waits until the bitmap step of the iteration with this tag has run: every word it writes for the host carries the tag, so that
// nothing else has to tell.  (An event behind it took the host 5 us, and the next kernel on the stream started 4 us later
// for it.)  What the caller has enqueued behind that step is not waited for: the words are looked at all the time for kLookUs, then
// every kSleepUs with the core given up in between; a look at the stream, every kStreamUs, is for errors and for a stream
// with nothing left to run.
int32_t await_bitmap(ddp_ctx* c, uint64_t tag) {
    constexpr int kLookUs = 1000, kSleepUs = 50, kStreamUs = 20000;
    using clock = std::chrono::steady_clock;
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    const auto sleep_from = clock::now() + std::chrono::microseconds(kLookUs);
    auto stream_from = clock::now() + std::chrono::microseconds(kStreamUs);
    for (int32_t g = 0; g < n; ++g)
        while (__atomic_load_n(c->h_global + g, __ATOMIC_ACQUIRE) >> 1 < tag) {
            const auto now = clock::now();
            if (now < sleep_from) continue;
            if (now >= stream_from) {
                const hipError_t q = hipStreamQuery(c->backward);
                if (q == hipSuccess) return DDP_OK;
                if (q != hipErrorNotReady) return fail(c, DDP_ERR_HIP, std::string("hipStreamQuery: ") + hipGetErrorString(q));
                stream_from = now + std::chrono::microseconds(kStreamUs);
            }
            std::this_thread::sleep_for(std::chrono::microseconds(kSleepUs));
        }
    return DDP_OK;
}

// Where a mask launch takes the masks of segments [begin, end) of the running iteration from: up to
// kMasksByValue go into kernel arguments, more are copied into pinned memory that the kernel reads.
// All kernels that read an iteration's copy are in front of its bitmap step, or are that step.
int32_t stage_masks(ddp_ctx* c, int begin, int end, const uint64_t** masks) {
    *masks = c->local_cur.data() + begin;
    if (end - begin <= ddp::kMasksByValue) return DDP_OK;
    const int par = static_cast<int>(c->iteration & 1);
    if (c->masks_claimed_iter != c->iteration) {
        if (c->masks_in_flight[par] != 0) {
            const int32_t rc = await_bitmap(c, c->masks_in_flight[par]);
            if (rc != DDP_OK) return rc;
        }
        c->masks_in_flight[par] = 0;
        c->masks_claimed_iter = c->iteration;
    }
    std::memcpy(c->h_masks[par] + begin, *masks, sizeof(uint64_t) * (end - begin));
    *masks = c->h_masks[par] + begin;
    return DDP_OK;
}

// Where a launch goes: a reduction stream taken in turn, the backward stream (the API call that
// completes the iteration, see flush_deferred), or the caller's reduction stream as the
// partner of the backward stream when such a call makes several launches.
enum class Target { kLane, kBackward, kPartner };

// Enqueue everything buckets [first, last] need, as one launch per kernel.  The buckets are
// consecutive, hold one element type, and their tiles and slab ranges are contiguous.
int32_t launch_range(ddp_ctx* c, int32_t first, int32_t last, Target target) {
    const ddp::BucketInfo& bf = c->plan.buckets[first];
    const ddp::BucketInfo& bl = c->plan.buckets[last];
    const int seg_begin = bf.seg_begin;
    const int seg_end = bl.seg_begin + static_cast<int>(bl.params.size());
    const int64_t tile_base = c->h_tile0[seg_begin];
    const int64_t ntiles = c->h_tile0[seg_end] - tile_base;
    const int64_t nslices = c->h_slices[seg_end] - c->h_slices[seg_begin];
    int64_t bytes = 0;
    for (int32_t b = first; b <= last; ++b) bytes += static_cast<int64_t>(c->plan.buckets[b].bytes());
    const int64_t traffic = launch_traffic(c, bytes);
    const int32_t id = first + 65536 * (last - first);
    int lane = -1;                    // -1: the backward stream
    hipStream_t st = c->backward;
    const bool may_be_early = target == Target::kLane && c->n_streams < 0 && c->tail_on_backward != 0 && traffic <= kEarlyTraffic &&
                              flags_usable(c);
    bool early = false;
    if (target == Target::kLane && c->n_streams < 0 && c->tail_on_backward != 0 && c->small_model) {
        // stays on the backward stream
    } else if (may_be_early && take_early(c, traffic)) {
        early = true;                 // ... and so does this launch
    } else if (target == Target::kLane) {
        // Short launches gain from a neighbour on a second stream (start-up and drain of one
        // overlap with the other); launches long enough for the cap on resident blocks lose
        // when two of them share the memory system, so by default those stay on one stream.
        const int lanes = c->n_streams < 0 ? (!long_launch(c, bytes) && c->lane[1] && c->lane_concurrent[1] ? 2 : 1) : c->n_streams;
        lane = static_cast<int>(c->launches_in_iter++ % lanes);
        // (short launches next to this one would take long to run: they look again first)
        if (traffic >= kChainMinTraffic) {
            c->early_credit = 0;
            c->progress_wait = 0;     // (an announcement in front of it says nothing of what comes behind)
        }
    } else if (target == Target::kPartner) {
        lane = 0;
    }
    if (lane >= 0 && c->lane[lane] != c->backward) {
        st = c->lane[lane];
        c->lane_used[lane] = true;
        c->latest_lane = lane;
    } else {
        lane = -1;
    }
    const ddp::GateRecord* gate = nullptr;
    ddp::DispatchSignal sig{nullptr, 0};
    if (lane >= 0 && (!c->lane_ordered[lane] || c->call_by_flag)) {
        const int32_t rc = order_call(c, first, may_be_early);
        if (rc != DDP_OK) return rc;
    }
    // Chained launches.  With flag ordering in use (so the streams are known to run side by
    // side and nothing is being captured), a launch that follows another launch of this
    // iteration on a DIFFERENT stream lets that one reach its last thread block first (a
    // bounded wait: in the gate of a launch on a reduction stream, in a one-wave kernel of its
    // own on the backward stream), so that the two overlap where one drains and the other
    // starts up rather than sharing the memory system all the way (on one stream, stream order
    // does more).  It pays from about 160 MiB moved by the launch in front (measured with one
    // mark per call, gain of chaining: 225 MiB +4.7 to +6.1 %, 170-180 MiB +3.2 to +5.4 %,
    // 125-135 MiB -1.2 to -3.0 %, 45-90 MiB -0.5 to -4.4 %: short launches are mostly start-up
    // and drain, and those overlap best when both run at once).  Two launches that are both
    // long enough for the cap on resident blocks are left alone: in turn on two streams,
    // chained, they lose 1.5 to 3 points against one stream (R = 16 and 32, binary32
    // outputs).  A launch on the backward stream is chained whenever it moves 160 MiB itself:
    // with back-to-back iterations it would otherwise run next to the iteration's first
    // launches for all of its time.  An early launch never is: what comes behind it on the backward stream
    // is the rest of the backward pass, which would wait for the launch in front of it too.
    const bool flags_in_use = c->call_by_flag || c->gates_in_iter > 0;
    const bool both_long = c->prev_launch_long && long_launch(c, bytes);
    const bool chained = c->chain_launches != 0 && flags_in_use && c->prev_launch_ord != 0 && c->prev_launch_lane != lane &&
                         ntiles > 0 && carries_gate(c) && !early &&
                         ((c->prev_launch_traffic >= kChainMinTraffic && !both_long) ||
                          (lane < 0 && traffic >= kChainMinTraffic));
    const long long wait_ticks = c->gate_wait_us * c->wall_clock_khz / 1000;
    c->tail_chained = lane < 0 && chained;
    if (lane < 0 && chained)
        HIPCHK(c, ddp::launch_chain_wait(c->d_order, c->prev_launch_ord, wait_ticks, st));
    if (lane >= 0 && (!c->lane_ordered[lane] || c->call_by_flag)) {
        if (c->call_by_flag) {
            // every launch gets a gate of its own: if the gate gives up, exactly this launch
            // is skipped and redone by the repair launch of the finalizing step
            if (c->gates_in_iter == 0 && c->iteration - c->safe_iteration >= ddp_ctx::kGateRows - 1) {
                // this iteration's row of gate records was last used kGateRows iterations ago:
                // that iteration's repair launch must have read it (a host that enqueues that
                // many iterations without ever synchronizing waits here once per cycle)
                HIPCHK(c, hipStreamSynchronize(c->backward));
                c->safe_iteration = c->iteration;
            }
            ddp::GateRecord* rec = c->gate_row() + first;
            HIPCHK(c, ddp::launch_gate(c->d_order, c->call_seq, wait_ticks, rec,
                                       c->gate_row() + c->plan.buckets.size(),
                                       static_cast<int32_t>(tile_base), static_cast<int32_t>(ntiles), bf.dtype,
                                       static_cast<uint32_t>(c->iteration + 1),
                                       chained ? c->prev_launch_ord : 0ull, chained ? wait_ticks : 0, st));
            gate = rec;
            ++c->gates_in_iter;
            look_at_progress(c);
        } else if (!c->backward_idle_in_call) {
            HIPCHK(c, hipStreamWaitEvent(st, c->call_event, 0));
        }
        c->lane_ordered[lane] = true;
    }
    if (c->chain_launches != 0 && (c->call_by_flag || c->gates_in_iter > 0) && ntiles > 0 && carries_gate(c)) {
        // the launch reports when its last block starts, for whatever is chained behind it
        sig.word = &c->d_order->dispatched;
        sig.ord = ++c->launch_ord;
        c->prev_launch_ord = sig.ord;
        c->prev_launch_lane = lane;
        c->prev_launch_traffic = traffic;
        c->prev_launch_long = long_launch(c, bytes);
    }
    // Participation masks travel to the device only for launches that hold a
    // zero bit (a replica that did not use a parameter, or a parameter nobody
    // marked); everything else runs without a mask table.
    ddp::Masks masks;
    uint64_t mask_words[ddp::kMaskWords];
    bool need_flags = false;
    for (int32_t b = first; b <= last; ++b) need_flags = need_flags || c->bucket_zero[b] != 0;
    const bool two_kernels = c->pipeline == DDP_PIPELINE_STAGED && (c->timing == 1 || split_pass(c, bf.dtype, ntiles, nslices));
    if (need_flags && !two_kernels && ddp::masks_fit(c->R, seg_end - seg_begin)) {
        ddp::pack_masks(c->local_cur.data() + seg_begin, seg_end - seg_begin, c->R, mask_words);
        masks.words = mask_words;
        masks.first = seg_begin;
    } else if (need_flags) {
        // After the ordering above the stream is also behind the previous iteration's readers of
        // the table (or its gate gave up and nothing is written).
        const uint64_t* host;
        const int32_t rcm = stage_masks(c, seg_begin, seg_end, &host);
        if (rcm != DDP_OK) return rcm;
        HIPCHK(c, ddp::launch_mask_write(c->d_local + seg_begin, host, seg_end - seg_begin,
                                         gate, static_cast<uint32_t>(c->iteration + 1), st));
        masks.table = c->d_local;
        look_at_progress(c);
    }
    const ddp::Scale sc = make_scale(c->R);
    size_t slot;
    int32_t rc;
    if (c->timing == 2 && c->open_group == static_cast<size_t>(-1)) {
        // one event pair per iteration: opened by its first bucket launch
        TimedLaunch t{DDP_K_ITERATION, 0, nullptr, nullptr};
        HIPCHK(c, hipEventCreateWithFlags(&t.start, kTimingEvent));
        HIPCHK(c, hipEventCreateWithFlags(&t.stop, kTimingEvent));
        HIPCHK(c, hipEventRecord(t.start, st));
        c->timed.push_back(t);
        c->open_group = c->timed.size() - 1;
    }
    if (c->timing == 2) c->timed[c->open_group].bucket += 1;   // counts the launches
    const uint32_t tag = static_cast<uint32_t>(c->iteration + 1);
    if (two_kernels) {
        // pack and reduce as launches of their own; timed one by one, each is stamped
        char* in0 = c->slabs + c->bucket_slab_off[first];
        char* out = c->slabs + static_cast<int64_t>(c->R) * c->slab_stride + c->bucket_slab_off[first];
        // the range of the slab from the first bucket's base to the last one's padded end
        const int64_t nvec = (c->bucket_slab_off[last] - c->bucket_slab_off[first]) / 16 + c->bucket_vecs[last];
        if ((rc = timed_begin(c, DDP_K_PACK, id, st, &slot)) != DDP_OK) return rc;
        HIPCHK(c, ddp::launch_pack(c->tables, tile_base, ntiles, c->slabs, c->slab_stride, c->R,
                                   masks.table, gate, tag, st));
        look_at_progress(c);
        if ((rc = timed_end(c, slot, st)) != DDP_OK) return rc;
        if ((rc = timed_begin(c, DDP_K_REDUCE, id, st, &slot)) != DDP_OK) return rc;
        HIPCHK(c, ddp::launch_flat_reduce(bf.dtype, in0, c->slab_stride, out, nvec, c->R, sc,
                                          c->nontemporal != 0,
                                          long_launch(c, bytes) ? occupancy_lds(c, bytes, ddp::elem_size(bf.dtype), false, need_flags) : 0, gate, tag, sig, st));
        if ((rc = timed_end(c, slot, st)) != DDP_OK) return rc;
    } else {
        const bool staged = c->pipeline == DDP_PIPELINE_STAGED;
        const ddp::FlatBuckets flat{staged ? c->slabs : nullptr, staged ? c->slab_stride : 0};
        if ((rc = timed_begin(c, DDP_K_REDUCE, id, st, &slot)) != DDP_OK) return rc;
        HIPCHK(c, ddp::launch_fused_reduce(bf.dtype, c->tables, tile_base, ntiles, c->h_slices[seg_begin], nslices, c->R,
                                           c->write_all ? c->R : 1, masks, c->find_unused != 0, sc,
                                           c->nontemporal != 0, occupancy_lds(c, bytes, ddp::elem_size(bf.dtype), staged, need_flags),
                                           flat, gate, tag, sig, st));
        if ((rc = timed_end(c, slot, st)) != DDP_OK) return rc;
    }
    look_at_progress(c);
    return DDP_OK;
}

// True if no replica used any parameter of bucket b in the running iteration.
bool bucket_all_unused(const ddp_ctx* c, int32_t b) {
    if (!c->bucket_zero[b]) return false;
    const ddp::BucketInfo& bk = c->plan.buckets[b];
    const size_t begin = static_cast<size_t>(bk.seg_begin);
    const size_t end = begin + bk.params.size();
    for (size_t k = begin; k < end; ++k)
        if (c->local_cur[k]) return false;
    return true;
}

// Enqueue the buckets the running API call has made launchable: one launch per
// bucket, or (DDP_OPT_COALESCE) one per run of consecutive buckets of equal
// element type.
int32_t flush_deferred(ddp_ctx* c) {
    if (c->deferred.empty()) return DDP_OK;
    std::vector<int32_t> todo;
    todo.swap(c->deferred);
    if (c->plan_only) return DDP_OK;
    HIPCHK(c, hipSetDevice(c->device));
    // Buckets are launched in index order, so if the last bucket is among the
    // ones this API call launches, every gradient of the iteration has been
    // produced and the backward stream has nothing left to overlap with.  The
    // call's launches then go to the backward stream: stream order replaces
    // the cross-stream event, whose hand-over costs about 0.2 ms here when the
    // waiting queue was armed long before the event fires.  (Staged pipeline: the write-back of the
    // finalizing step follows on the same stream.  ResNet-50, R = 8, all marks in one call: 375 us a
    // synchronization with the launches and the write-back on the reduction stream, 348 so; the eight
    // small tensors in one bucket, R = 2: 46 and 8 us.)
    const bool closing = c->tail_on_backward != 0 &&
                         todo.back() == static_cast<int32_t>(c->plan.buckets.size()) - 1;
    if (c->find_unused != 0 && c->pipeline == DDP_PIPELINE_FUSED && c->iter_zero) {
        // Skipping at the bucket level (Section 6.2.2): a bucket none of whose
        // parameters was used by any replica has nothing to reduce and, with
        // find_unused, nothing to write -- it needs no launch at all.
        size_t kept = 0;
        for (int32_t b : todo)
            if (!bucket_all_unused(c, b)) todo[kept++] = b;
        todo.resize(kept);
        if (todo.empty()) return DDP_OK;
    }
    std::vector<std::pair<int32_t, int32_t>> ranges;      // [first, last] bucket of every launch
    size_t i = 0;
    while (i < todo.size()) {
        size_t j = i;
        const int64_t limit = launch_limit(c);
        if (limit > 0) {
            // the run of consecutive buckets of one type that starts here, as far as a last launch reaches
            const uint64_t most = static_cast<uint64_t>(last_launch_limit(c));
            size_t end = i + 1;
            uint64_t bytes = c->plan.buckets[todo[i]].bytes(), run = bytes;
            while (end < todo.size() && run <= most && todo[end] == todo[end - 1] + 1 &&
                   c->plan.buckets[todo[end]].dtype == c->plan.buckets[todo[i]].dtype)
                run += c->plan.buckets[todo[end++]].bytes();
            if (run <= most) j = end - 1;
            else
                while (j + 1 < end && bytes + c->plan.buckets[todo[j + 1]].bytes() <= static_cast<uint64_t>(limit))
                    bytes += c->plan.buckets[todo[++j]].bytes();
        }
        ranges.emplace_back(todo[i], todo[j]);
        i = j + 1;
    }
    // A closing call that makes several launches: on one stream each launch would start when
    // the one before has drained.  With chained launches they take the backward stream and the
    // caller's reduction stream in turn instead, every launch starting as its predecessor
    // reaches its last thread block.  The announcement that orders the reduction stream's
    // share goes out first, ahead of the backward stream's own launches.
    bool partner = false;
    if (closing && ranges.size() > 1 && c->chain_launches != 0 && c->reduce != c->backward && flags_usable(c)) {
        const int32_t rc = order_call(c, ranges[0].first, false);
        if (rc != DDP_OK) return rc;
        partner = c->call_by_flag;
    }
    bool prev_on_backward = false, prev_long = false;
    for (size_t k = 0; k < ranges.size(); ++k) {
        int64_t bytes = 0;
        for (int32_t b = ranges[k].first; b <= ranges[k].second; ++b) bytes += static_cast<int64_t>(c->plan.buckets[b].bytes());
        // Two launches that both move as much as a long one do best one after the other on one stream.
        // (Staged, 2 R + 1 times the bucket bytes: the first 101 BERT-large tensors, R = 2, 400 MiB and
        // 100, 520 us with the second on the partner, 501 so; 140 tensors, R = 8, 1908 and 1878.)
        const bool is_long = launch_traffic(c, bytes) >= c->cap_min_traffic;
        const bool to_partner = partner && k > 0 && prev_on_backward && !(prev_long && is_long);
        const Target target = !closing ? Target::kLane : to_partner ? Target::kPartner : Target::kBackward;
        const int32_t st = launch_range(c, ranges[k].first, ranges[k].second, target);
        if (st != DDP_OK) return st;
        prev_on_backward = target == Target::kBackward;
        prev_long = is_long;
    }
    return DDP_OK;
}

// Bucket b has become launchable: log it and queue it for flush_deferred.
void note_launch(ddp_ctx* c, int32_t b, int32_t call_index) {
    c->log_running.emplace_back(b, call_index);
    c->deferred.push_back(b);
}

// Frees what ddp_build_buckets allocates (also after a build that failed half
// way, so that a retry does not leak).
void release_build(ddp_ctx* c) {
    for (hipEvent_t e : c->ev_ready)
        if (e) (void)hipEventDestroy(e);
    c->ev_ready.clear();
    if (c->slabs) (void)hipFree(c->slabs);
    if (c->d_tables) (void)hipFree(c->d_tables);
    if (c->d_tile_seg) (void)hipFree(c->d_tile_seg);
    if (c->d_local) (void)hipFree(c->d_local);
    if (c->d_global) (void)hipFree(c->d_global);
    if (c->d_micro) (void)hipFree(c->d_micro);
    if (c->d_gate) (void)hipFree(c->d_gate);
    c->d_gate = nullptr;
    if (c->h_global) (void)hipHostFree(c->h_global);
    for (uint64_t*& m : c->h_masks) {
        if (m) (void)hipHostFree(m);
        m = nullptr;
    }
    if (c->h_micro) (void)hipHostFree(c->h_micro);
    c->slabs = nullptr; c->d_tables = nullptr; c->d_tile_seg = nullptr; c->d_local = nullptr;
    c->d_global = nullptr; c->d_micro = nullptr; c->h_global = nullptr; c->h_micro = nullptr;
}

void release_device(ddp_ctx* c) {
    if (c->plan_only) return;
    (void)hipSetDevice(c->device);
    bool ended = true;                 // nothing of the context is under way
    auto wait = [&](hipStream_t s) { ended = hipStreamSynchronize(s) == hipSuccess && ended; };
    if (c->reduce) wait(c->reduce);
    if (c->backward) wait(c->backward);
    if (!c->reduce || !c->backward) wait(nullptr);
    for (int l = 1; l < ddp_ctx::kMaxLanes; ++l) {
        if (c->lane[l]) {
            wait(c->lane[l]);
            (void)hipStreamDestroy(c->lane[l]);
            c->lane[l] = nullptr;
        }
        if (c->ev_join[l]) { (void)hipEventDestroy(c->ev_join[l]); c->ev_join[l] = nullptr; }
    }
    for (uint64_t*& w : c->done_word) {
        if (w && ended) give_word(c->device, w);      // (else it is left alone: a kernel may still write it)
        w = nullptr;
    }
    drop_timed(c);
    release_build(c);
    for (hipEvent_t* e : {&c->ev_done, &c->ev_emit})
        if (*e) { (void)hipEventDestroy(*e); *e = nullptr; }
    if (c->d_order_mem) (void)hipFree(c->d_order_mem);
    c->d_order_mem = nullptr; c->d_order = nullptr; c->d_probe = nullptr;
    if (c->h_progress) (void)hipHostFree(c->h_progress);
    c->h_progress = nullptr;
    if (c->d_emit) (void)hipFree(c->d_emit);
    if (c->h_emit) (void)hipHostFree(c->h_emit);
    c->d_emit = nullptr; c->h_emit = nullptr;
}

inline int64_t round_up(int64_t x, int64_t a) { return ddp::round_up_to(x, a); }

}  // namespace

namespace ddp {
int32_t fail_without_context(int32_t code, const std::string& msg) { return fail(nullptr, code, msg); }
}  // namespace ddp

extern "C" {

#ifndef DDP_SOURCE_HASH
#define DDP_SOURCE_HASH "0000000000000000"
#endif
// The build passes a digest of the sources; the Python binding compares it with
// the sources on disk so that a stale library is never tested or measured.
const char* ddp_version(void) { return "ddp_gfx950 0.2 ddp-src-hash:" DDP_SOURCE_HASH; }

const char* ddp_last_error(const ddp_ctx* ctx) {
    return ctx ? ctx->err.c_str() : g_create_error.c_str();
}

int32_t ddp_create(ddp_ctx** out, int32_t R, int32_t device, void* reduce_stream,
                   void* backward_stream) {
    if (!out) return fail(nullptr, DDP_ERR_ARG, "ddp_create: out is null");
    *out = nullptr;
    if (R < 1) return fail(nullptr, DDP_ERR_ARG, "ddp_create: R must be at least 1");
    if (R > DDP_MAX_REPLICAS) return fail(nullptr, DDP_ERR_UNSUPPORTED, "ddp_create: R above DDP_MAX_REPLICAS");
    if (device < DDP_DEVICE_NONE) return fail(nullptr, DDP_ERR_ARG, "ddp_create: bad device");
    ddp_ctx* c = new ddp_ctx();
    c->R = R;
    c->device = device;
    c->plan_only = device == DDP_DEVICE_NONE;
    c->reduce = static_cast<hipStream_t>(reduce_stream);
    c->backward = static_cast<hipStream_t>(backward_stream);
    c->lane[0] = c->reduce;
    if (!c->plan_only) {
        int count = 0;
        hipError_t e = hipGetDeviceCount(&count);
        if (e != hipSuccess || device >= count) {
            delete c;
            return fail(nullptr, DDP_ERR_HIP, "ddp_create: no such HIP device (the library needs a GPU; "
                                              "use DDP_DEVICE_NONE only for plan inspection)");
        }
        e = hipSetDevice(device);
        int khz = 0;
        if (e == hipSuccess) e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device);
        if (e == hipSuccess && khz > 0) c->wall_clock_khz = khz;
        int lds = 0;
        if (e == hipSuccess) e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, device);
        if (e == hipSuccess && lds >= 64 * 1024) c->lds_per_cu = lds;
        if (e == hipSuccess) e = hipEventCreateWithFlags(&c->ev_done, kOrderEvent);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&c->ev_emit, hipEventDisableTiming);
        int cus = 0;
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
        if (e == hipSuccess && cus > 0) c->num_cus = cus;
        const size_t order_bytes = sizeof(ddp::OrderState) + 3 * sizeof(unsigned long long);
        if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&c->d_order_mem), order_bytes);
        if (e == hipSuccess) e = hipMemset(c->d_order_mem, 0, order_bytes);
        if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&c->h_progress), sizeof(unsigned long long), hipHostMallocDefault);
        if (e == hipSuccess) *c->h_progress = 0;
        if (e == hipSuccess) e = hipDeviceSynchronize();
        if (e != hipSuccess) {
            std::string msg = std::string("ddp_create: ") + hipGetErrorString(e);
            release_device(c);
            delete c;
            return fail(nullptr, DDP_ERR_HIP, msg);
        }
        c->d_order = reinterpret_cast<ddp::OrderState*>(c->d_order_mem);
        c->d_probe = reinterpret_cast<unsigned long long*>(c->d_order_mem + sizeof(ddp::OrderState));
        // the second reduction stream of the default configuration (not when both roles share
        // one stream: then nothing can overlap anyway)
        if (probe_lane(c, 0) != DDP_OK || (c->reduce != c->backward && create_lane(c, 1) != DDP_OK)) {
            std::string msg = "ddp_create: stream probe: " + c->err;
            release_device(c);
            delete c;
            return fail(nullptr, DDP_ERR_HIP, msg);
        }
    }
    *out = c;
    return DDP_OK;
}

int32_t ddp_destroy(ddp_ctx* ctx) {
    if (!ctx) return DDP_ERR_ARG;
    release_device(ctx);
    delete ctx;
    return DDP_OK;
}

int32_t ddp_set_option(ddp_ctx* c, int32_t option, int64_t value) {
    if (!c) return DDP_ERR_ARG;
    switch (option) {
        case DDP_OPT_PIPELINE:
            if (c->built) return fail(c, DDP_ERR_STATE, "pipeline must be chosen before ddp_build_buckets");
            if (value != DDP_PIPELINE_STAGED && value != DDP_PIPELINE_FUSED)
                return fail(c, DDP_ERR_ARG, "unknown pipeline");
            c->pipeline = static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_WRITE_ALL:
            if (c->built) return fail(c, DDP_ERR_STATE, "write-all must be chosen before ddp_build_buckets");
            c->write_all = value != 0;
            return DDP_OK;
        case DDP_OPT_TIMING:
            if (!c->plan_only) {
                (void)hipSetDevice(c->device);
                drop_timed(c);
            }
            if (value < 0 || value > 2) return fail(c, DDP_ERR_ARG, "timing mode must be 0, 1 or 2");
            c->timing = c->plan_only ? 0 : static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_EMIT_BUSY_BLOCKS:
            if (value < 0 || value > 4096) return fail(c, DDP_ERR_ARG, "busy blocks outside [0, 4096]");
            c->emit_busy_blocks = static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_FIND_UNUSED:
            c->find_unused = value != 0;
            return DDP_OK;
        case DDP_OPT_REDUCE_BLOCKS_PER_CU:
            if (value < -1 || value > 16) return fail(c, DDP_ERR_ARG, "blocks per compute unit outside [-1, 16]");
            c->blocks_per_cu = static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_ACCUMULATE_BLOCKS_PER_CU:
            if (value < -1 || value > 16) return fail(c, DDP_ERR_ARG, "blocks per compute unit outside [-1, 16]");
            c->acc_blocks_per_cu = static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_REDUCE_CAP_MIN_BYTES:
            if (value < 0) return fail(c, DDP_ERR_ARG, "bad size");
            c->cap_min_traffic = value;
            c->cap_min_set = true;
            return DDP_OK;
        case DDP_OPT_TAIL_ON_BACKWARD:
            c->tail_on_backward = value != 0;
            return DDP_OK;
        case DDP_OPT_REDUCE_STREAMS:
            if (value != -1 && (value < 1 || value > ddp_ctx::kMaxLanes))
                return fail(c, DDP_ERR_ARG, "number of reduction streams outside [1, 8] and not -1");
            if (c->tracker.marks() != 0 || !c->log_running.empty())
                return fail(c, DDP_ERR_STATE, "reduction streams can only change between iterations");
            if (!c->plan_only) {
                HIPCHK(c, hipSetDevice(c->device));
                for (int l = 1; l < value; ++l) {
                    const int32_t rc = create_lane(c, l);
                    if (rc != DDP_OK) return rc;
                }
            }
            c->n_streams = static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_LAUNCH_HOLD:
            if (value < 0 || value > 1000000) return fail(c, DDP_ERR_ARG, "launch hold outside [0, 1000000] marks");
            if (c->tracker.marks() != 0 || !c->log_running.empty())
                return fail(c, DDP_ERR_STATE, "the launch hold can only change between iterations");
            c->hold_marks = static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_FLAG_ORDER:
            if (value != -1 && value != 0) return fail(c, DDP_ERR_ARG, "flag ordering must be -1 (where possible) or 0 (never)");
            if (c->tracker.marks() != 0 || !c->log_running.empty())
                return fail(c, DDP_ERR_STATE, "the ordering mode can only change between iterations");
            c->flag_order = static_cast<int32_t>(value);
            return DDP_OK;
        case DDP_OPT_CHAIN_LAUNCHES:
            c->chain_launches = value != 0;
            return DDP_OK;
        case DDP_OPT_GATE_WAIT_US:
            if (value < 0 || value > 10000000) return fail(c, DDP_ERR_ARG, "gate wait outside [0, 10 s]");
            c->gate_wait_us = value;
            return DDP_OK;
        case DDP_OPT_COALESCE:
            if (value < -1) return fail(c, DDP_ERR_ARG, "bad size");
            c->coalesce = value;
            return DDP_OK;
        case DDP_OPT_NONTEMPORAL:
            c->nontemporal = value != 0;
            return DDP_OK;
        default:
            return fail(c, DDP_ERR_ARG, "unknown option");
    }
}

int32_t ddp_get_option(ddp_ctx* c, int32_t option, int64_t* value) {
    if (!c || !value) return DDP_ERR_ARG;
    switch (option) {
        case DDP_STAT_REPAIRED_LAUNCHES: {
            *value = 0;
            if (c->plan_only) return DDP_OK;
            HIPCHK(c, hipSetDevice(c->device));
            const int32_t rc = ddp_synchronize(c);
            if (rc != DDP_OK) return rc;
            uint32_t n = 0;
            HIPCHK(c, hipMemcpy(&n, &c->d_order->repaired, sizeof(n), hipMemcpyDeviceToHost));
            *value = n;
            return DDP_OK;
        }
        case DDP_STAT_EARLY_LAUNCHES: *value = c->early_total; return DDP_OK;
        case DDP_OPT_PIPELINE: *value = c->pipeline; return DDP_OK;
        case DDP_OPT_WRITE_ALL: *value = c->write_all; return DDP_OK;
        case DDP_OPT_TIMING: *value = c->timing; return DDP_OK;
        case DDP_OPT_FIND_UNUSED: *value = c->find_unused; return DDP_OK;
        case DDP_OPT_REDUCE_STREAMS: *value = c->n_streams; return DDP_OK;
        case DDP_OPT_COALESCE: *value = launch_limit(c); return DDP_OK;
        case DDP_OPT_TAIL_ON_BACKWARD: *value = c->tail_on_backward; return DDP_OK;
        case DDP_OPT_GATE_WAIT_US: *value = c->gate_wait_us; return DDP_OK;
        case DDP_OPT_LAUNCH_HOLD: *value = c->hold_marks; return DDP_OK;
        case DDP_OPT_FLAG_ORDER: *value = flags_usable(c) ? 1 : 0; return DDP_OK;
        case DDP_OPT_CHAIN_LAUNCHES: *value = c->chain_launches; return DDP_OK;
        case DDP_OPT_NONTEMPORAL: *value = c->nontemporal; return DDP_OK;
        case DDP_OPT_EMIT_BUSY_BLOCKS: *value = c->emit_busy_blocks; return DDP_OK;
        case DDP_OPT_REDUCE_BLOCKS_PER_CU: *value = c->blocks_per_cu; return DDP_OK;
        case DDP_OPT_REDUCE_CAP_MIN_BYTES: *value = c->cap_min_traffic; return DDP_OK;
        case DDP_OPT_ACCUMULATE_BLOCKS_PER_CU: *value = c->acc_blocks_per_cu; return DDP_OK;
        default: return fail(c, DDP_ERR_ARG, "unknown option");
    }
}

int32_t ddp_register_params(ddp_ctx* c, int32_t n, const int64_t* numel, const int32_t* dtype,
                            void* const* grad_ptrs) {
    if (!c) return DDP_ERR_ARG;
    if (c->registered) return fail(c, DDP_ERR_STATE, "ddp_register_params called twice");
    if (n <= 0 || !numel || !dtype) return fail(c, DDP_ERR_ARG, "ddp_register_params: n <= 0 or null array");
    if (!c->plan_only && !grad_ptrs) return fail(c, DDP_ERR_ARG, "ddp_register_params: grad_ptrs is null");
    for (int32_t i = 0; i < n; ++i) {
        if (numel[i] < 0) return fail(c, DDP_ERR_ARG, "ddp_register_params: negative numel");
        if (dtype[i] != DDP_FP32 && dtype[i] != DDP_FP16 && dtype[i] != DDP_BF16)
            return fail(c, DDP_ERR_ARG, "ddp_register_params: unknown dtype");
    }
    if (!c->plan_only) {
        for (int32_t r = 0; r < c->R; ++r)
            for (int32_t i = 0; i < n; ++i) {
                const void* p = grad_ptrs[static_cast<int64_t>(r) * n + i];
                if (numel[i] > 0 && !p) return fail(c, DDP_ERR_ARG, "ddp_register_params: null gradient pointer");
                if (reinterpret_cast<uintptr_t>(p) % static_cast<uintptr_t>(ddp::elem_size(dtype[i])) != 0)
                    return fail(c, DDP_ERR_ARG, "ddp_register_params: gradient pointer not aligned to its element size");
            }
        c->grad_ptrs.assign(grad_ptrs, grad_ptrs + static_cast<int64_t>(c->R) * n);
    }
    c->plan.params.resize(n);
    for (int32_t i = 0; i < n; ++i) {
        c->plan.params[i].numel = numel[i];
        c->plan.params[i].dtype = dtype[i];
    }
    c->registered = true;
    return DDP_OK;
}

int32_t ddp_set_outputs(ddp_ctx* c, void* const* out_ptrs) {
    if (!c) return DDP_ERR_ARG;
    if (!c->registered) return fail(c, DDP_ERR_STATE, "ddp_set_outputs before ddp_register_params");
    if (c->built) return fail(c, DDP_ERR_STATE, "ddp_set_outputs after ddp_build_buckets");
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    for (int32_t i = 0; i < n; ++i)
        if (c->plan.params[i].dtype != DDP_FP16 && c->plan.params[i].dtype != DDP_BF16)
            return fail(c, DDP_ERR_ARG, "ddp_set_outputs: binary32 outputs are for gradients held in fp16 or bf16");
    if (c->plan_only) {            // the plan does not depend on where the averages go
        c->out_ptrs.assign(n, nullptr);
        return DDP_OK;
    }
    if (!out_ptrs) return fail(c, DDP_ERR_ARG, "ddp_set_outputs: out_ptrs is null");
    for (int32_t i = 0; i < n; ++i) {
        if (c->plan.params[i].numel > 0 && !out_ptrs[i]) return fail(c, DDP_ERR_ARG, "ddp_set_outputs: null output pointer");
        if (reinterpret_cast<uintptr_t>(out_ptrs[i]) % 4 != 0)
            return fail(c, DDP_ERR_ARG, "ddp_set_outputs: output pointer not aligned to 4 bytes");
    }
    c->out_ptrs.assign(out_ptrs, out_ptrs + n);
    return DDP_OK;
}

// Assigns the buckets (visiting the parameters in `order`, or in reverse
// registration order without one) and builds everything that depends on the
// assignment: tracker, flag tables, slabs, segment tables, events.
static int32_t build_internal(ddp_ctx* c, uint64_t cap_bytes, const std::vector<int32_t>* order) {
    if (!c->plan.assign(cap_bytes, order)) return fail(c, DDP_ERR_ARG, "visit order is not a permutation");
    c->tracker.reset(c->plan);
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    const int32_t nb = static_cast<int32_t>(c->plan.buckets.size());
    c->used_running.assign(n, 0);
    c->used_closed.assign(n, 0);
    c->local_cur.assign(n, 0);
    c->acc_used.assign(n, 0);
    c->micro_used.assign(n, 0);
    c->bucket_zero.assign(nb, 0);
    c->global_closed.assign(n, 0);

    c->wide = false;
    for (const ddp::BucketInfo& bk : c->plan.buckets) c->wide = c->wide || bk.dtype == DDP_FP32;
    int64_t total_bytes = 0;
    for (const ddp::BucketInfo& bk : c->plan.buckets) total_bytes += static_cast<int64_t>(bk.bytes());
    c->small_model = nb <= kSmallModelBuckets && int64_t(c->R) * (nb - 1) <= kSmallModelReplicas &&
                     total_bytes < kSmallModelTraffic &&
                     launch_traffic(c, total_bytes) < kSmallModelTraffic;

    if (!c->plan_only) {
        // slab layout (bucket bases aligned to 256 bytes, lengths padded to 16) and segment
        // tables in bucket-major fill order
        ddp::HostTables ht;
        if (!c->out_ptrs.empty()) {
            if (c->pipeline != DDP_PIPELINE_FUSED)
                return fail(c, DDP_ERR_UNSUPPORTED, "binary32 outputs (ddp_set_outputs) need the fused pipeline");
            if (c->write_all)
                return fail(c, DDP_ERR_UNSUPPORTED, "binary32 outputs (ddp_set_outputs) cannot be combined with DDP_OPT_WRITE_ALL");
        }
        ddp::build_host_tables(c->plan, c->grad_ptrs.data(), c->R, ht, c->out_ptrs.empty() ? nullptr : c->out_ptrs.data(), true);
        c->bucket_slab_off = ht.bucket_slab_off;
        c->bucket_vecs = ht.bucket_vecs;
        c->slab_stride = ht.slab_stride;
        c->h_tile0 = ht.tile0;
        c->h_slices = ht.slices;
        if (c->h_tile0[n] >= (int64_t(1) << 31)) {
            c->built = false;
            return fail(c, DDP_ERR_UNSUPPORTED, "model too large for one launch grid");
        }
        HIPCHK(c, hipSetDevice(c->device));
        release_build(c);   // leftovers of an earlier attempt that failed
        // one allocation for the segment records and the pointer rows
        const int64_t R = c->R;
        const size_t seg_bytes = sizeof(ddp::SegInfo) * n;
        const size_t grad_bytes = sizeof(void*) * ht.grad.size();
        const size_t bytes = seg_bytes + grad_bytes + sizeof(void*) * ht.out.size();
        std::vector<char> host(bytes);
        std::memcpy(host.data(), ht.seg.data(), seg_bytes);
        std::memcpy(host.data() + seg_bytes, ht.grad.data(), grad_bytes);
        if (!ht.out.empty()) std::memcpy(host.data() + seg_bytes + grad_bytes, ht.out.data(), sizeof(void*) * ht.out.size());
        HIPCHK(c, hipMalloc(&c->d_tables, bytes));
        HIPCHK(c, hipMemcpy(c->d_tables, host.data(), bytes, hipMemcpyHostToDevice));
        char* d = static_cast<char*>(c->d_tables);
        c->tables.seg = reinterpret_cast<const ddp::SegInfo*>(d);
        c->tables.grad = reinterpret_cast<void* const*>(d + seg_bytes);
        c->tables.out = ht.out.empty() ? nullptr : reinterpret_cast<void* const*>(d + seg_bytes + grad_bytes);
        c->tables.G = n;
        c->tables.R = c->R;
        {
            const std::vector<int32_t>& tile_seg = ht.tile_seg;
            const size_t tb = sizeof(int32_t) * (tile_seg.empty() ? 1 : tile_seg.size());
            HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->d_tile_seg), tb));
            if (!tile_seg.empty())
                HIPCHK(c, hipMemcpy(c->d_tile_seg, tile_seg.data(), sizeof(int32_t) * tile_seg.size(), hipMemcpyHostToDevice));
            c->tables.tile_seg = c->d_tile_seg;
            c->tables.slices = ht.listed ? c->d_tile_seg + c->h_tile0[n] : nullptr;
        }

        HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->d_local), sizeof(uint64_t) * n));
        HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->d_global), static_cast<size_t>(n) + 16));
        HIPCHK(c, hipHostMalloc(reinterpret_cast<void**>(&c->h_global), sizeof(uint64_t) * n, hipHostMallocDefault));
        std::memset(c->h_global, 0, sizeof(uint64_t) * n);
        if (n > ddp::kMasksByValue)
            for (uint64_t*& m : c->h_masks)
                HIPCHK(c, hipHostMalloc(reinterpret_cast<void**>(&m), sizeof(uint64_t) * n, hipHostMallocDefault));
        c->micro_table = round_up(R * n, 2);
        const size_t micro_bytes = sizeof(void*) * static_cast<size_t>(c->micro_table);
        c->micro_slots = micro_bytes <= ddp_ctx::kSmallMicroTable ? 4 : 2;
        const size_t pinned_bytes = micro_bytes * static_cast<size_t>(c->micro_slots) + sizeof(unsigned long long);
        HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->d_micro), micro_bytes + sizeof(unsigned long long)));
        HIPCHK(c, hipMemset(c->d_micro + c->micro_table, 0, sizeof(unsigned long long)));
        HIPCHK(c, hipHostMalloc(reinterpret_cast<void**>(&c->h_micro), pinned_bytes, hipHostMallocDefault));
        std::memset(c->h_micro, 0, pinned_bytes);
        c->micro_ticket = 0;
        HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->d_gate), sizeof(ddp::GateRecord) * (nb + 1) * ddp_ctx::kGateRows));
        HIPCHK(c, hipMemset(c->d_gate, 0, sizeof(ddp::GateRecord) * (nb + 1) * ddp_ctx::kGateRows));
        c->gates_in_iter = 0;
        c->safe_iteration = c->iteration;
        c->ev_ready.resize(nb, nullptr);
        for (int32_t b = 0; b < nb; ++b)
            HIPCHK(c, hipEventCreateWithFlags(&c->ev_ready[b], kOrderEvent));
        if (c->pipeline == DDP_PIPELINE_STAGED) {
            const size_t total = static_cast<size_t>(c->slab_stride) * static_cast<size_t>(R + 1);
            HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->slabs), total));
            HIPCHK(c, hipMemset(c->slabs, 0, total));
        }
        HIPCHK(c, hipDeviceSynchronize());
    }
    c->built = true;
    return nb;
}

int32_t ddp_build_buckets(ddp_ctx* c, uint64_t cap_bytes) {
    if (!c) return DDP_ERR_ARG;
    if (!c->registered) return fail(c, DDP_ERR_STATE, "ddp_build_buckets before ddp_register_params");
    if (c->built) return fail(c, DDP_ERR_STATE, "ddp_build_buckets called twice");
    return build_internal(c, cap_bytes, nullptr);
}

int32_t ddp_rebuild_buckets(ddp_ctx* c, uint64_t cap_bytes) {
    if (!c) return DDP_ERR_ARG;
    if (!c->built) return fail(c, DDP_ERR_STATE, "ddp_rebuild_buckets before ddp_build_buckets");
    if (c->tracker.marks() != 0 || !c->deferred.empty())
        return fail(c, DDP_ERR_STATE, "ddp_rebuild_buckets in the middle of an iteration");
    for (uint64_t u : c->acc_used)
        if (u) return fail(c, DDP_ERR_STATE, "ddp_rebuild_buckets between a no_sync accumulation and its synchronization");
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    // visit order: the trace of the closed iteration, then what it never saw in
    // reverse registration order
    std::vector<int32_t> order = c->order_closed;
    {
        std::vector<uint8_t> seen(n, 0);
        for (int32_t p : order) seen[p] = 1;
        for (int32_t i = n - 1; i >= 0; --i)
            if (!seen[i]) order.push_back(i);
    }
    if (!c->plan_only) {
        // nothing may still use the tables, slabs and staging buffers that are about to be freed
        HIPCHK(c, hipSetDevice(c->device));
        HIPCHK(c, hipStreamSynchronize(c->backward));
        for (int l = 1; l < ddp_ctx::kMaxLanes; ++l)
            if (c->lane[l]) HIPCHK(c, hipStreamSynchronize(c->lane[l]));
        HIPCHK(c, hipStreamSynchronize(c->reduce));
        if (c->global_on_device) {      // keep the closed iteration's bitmap readable
            for (int32_t i = 0; i < n; ++i) c->global_closed[i] = c->h_global[c->plan.params[i].segment] & 1;
            c->global_on_device = false;
        }
        drop_timed(c);
        c->masks_in_flight[0] = c->masks_in_flight[1] = 0;
        c->masks_claimed_iter = -1;
    }
    const std::vector<uint8_t> keep_global = c->global_closed, keep_used = c->used_closed;
    c->built = false;
    const int32_t nb = build_internal(c, cap_bytes, &order);
    if (nb < 0) return nb;
    c->global_closed = keep_global;     // indexed by parameter: unaffected by the new mapping
    c->used_closed = keep_used;
    c->log_closed.clear();              // its bucket numbers belong to the old mapping
    return nb;
}

int32_t ddp_get_ready_order(const ddp_ctx* c, int32_t which, int32_t* ids, int32_t cap, int32_t* n) {
    if (!c || !n || cap < 0 || (which != 0 && which != 1)) return DDP_ERR_ARG;
    if (!c->built) return DDP_ERR_STATE;
    const std::vector<int32_t>& o = which == 0 ? c->order_running : c->order_closed;
    *n = static_cast<int32_t>(o.size());
    for (int32_t i = 0; i < *n && i < cap; ++i)
        if (ids) ids[i] = o[i];
    return DDP_OK;
}

int32_t ddp_get_assignment(const ddp_ctx* c, int32_t* bucket_of, int64_t* elem_offset) {
    if (!c || !bucket_of || !elem_offset) return DDP_ERR_ARG;
    if (!c->built) return DDP_ERR_STATE;
    for (size_t i = 0; i < c->plan.params.size(); ++i) {
        bucket_of[i] = c->plan.params[i].bucket;
        elem_offset[i] = c->plan.params[i].offset;
    }
    return DDP_OK;
}

int32_t ddp_get_bucket_info(const ddp_ctx* c, int32_t b, int64_t* elems, int32_t* n_params,
                            int32_t* dtype) {
    if (!c) return DDP_ERR_ARG;
    if (!c->built) return DDP_ERR_STATE;
    if (b < 0 || b >= static_cast<int32_t>(c->plan.buckets.size())) return DDP_ERR_ARG;
    const ddp::BucketInfo& bk = c->plan.buckets[b];
    if (elems) *elems = bk.elems;
    if (n_params) *n_params = static_cast<int32_t>(bk.params.size());
    if (dtype) *dtype = bk.dtype;
    return DDP_OK;
}

int32_t ddp_get_bucket_ptr(const ddp_ctx* c, int32_t b, int32_t r, void** ptr) {
    if (!c || !ptr) return DDP_ERR_ARG;
    if (!c->built) return DDP_ERR_STATE;
    if (c->plan_only) return DDP_ERR_NO_DEVICE;
    if (c->pipeline != DDP_PIPELINE_STAGED || !c->slabs) return DDP_ERR_STATE;
    if (b < 0 || b >= static_cast<int32_t>(c->plan.buckets.size()) || r < -1 || r >= c->R) return DDP_ERR_ARG;
    const int64_t slab = r < 0 ? c->R : r;
    *ptr = c->slabs + slab * c->slab_stride + c->bucket_slab_off[b];
    return DDP_OK;
}

static uint64_t everyone_mask(const ddp_ctx* c) { return c->R >= 64 ? ~uint64_t(0) : (uint64_t(1) << c->R) - 1; }

// Writes the participation mask of a parameter: `used`, OR what no_sync
// iterations recorded.  Returns whether any replica used it.
static bool set_participation(ddp_ctx* c, int32_t param_id, uint64_t used) {
    const ddp::ParamInfo& p = c->plan.params[param_id];
    const uint64_t eff = used | c->acc_used[p.segment];
    c->local_cur[p.segment] = eff;
    if (eff != everyone_mask(c)) {
        c->bucket_zero[p.bucket] = 1;
        c->iter_zero = true;
    }
    return eff != 0;
}

// What a single ready-mark call does with the buckets that are launchable: enqueue them now
// (the default: Algorithm 1 launches a bucket as soon as it is ready), or, with
// DDP_OPT_LAUNCH_HOLD, keep them back for a bounded number of further marks so that buckets
// that become ready shortly afterwards share their launch.
static int32_t flush_or_hold(ddp_ctx* c) {
    if (c->deferred.empty() || c->hold_marks <= 0) return flush_deferred(c);
    const int32_t last = static_cast<int32_t>(c->plan.buckets.size()) - 1;
    bool now = c->deferred.back() == last || c->tracker.marks() >= c->hold_until;
    if (!now) {
        uint64_t bytes = 0;
        for (int32_t b : c->deferred) bytes += c->plan.buckets[b].bytes();
        const int64_t limit = coalesce_limit(c);
        now = limit <= 0 || bytes >= static_cast<uint64_t>(limit);     // nothing more fits into the launch
    }
    return now ? flush_deferred(c) : DDP_OK;
}

static int32_t mark_one(ddp_ctx* c, int32_t param_id, uint64_t used) {
    std::vector<int32_t> launch;
    const int rc = c->tracker.mark(param_id, launch);
    if (rc == -1) return fail(c, DDP_ERR_ARG, "ddp_mark_ready: parameter id out of range");
    if (rc == -2) return fail(c, DDP_ERR_ALREADY_READY, "ddp_mark_ready: parameter already marked in this iteration");
    c->order_running.push_back(param_id);
    if (set_participation(c, param_id, used)) c->used_running[param_id] = 1;
    for (int32_t b : launch) note_launch(c, b, c->tracker.marks() - 1);
    if (!launch.empty()) c->hold_until = c->tracker.marks() + c->hold_marks;
    if (coalesce_limit(c) <= 0) return flush_deferred(c);
    return DDP_OK;
}

int32_t ddp_mark_ready(ddp_ctx* c, int32_t param_id) {
    if (!c) return DDP_ERR_ARG;
    if (!c->built) return fail(c, DDP_ERR_STATE, "ddp_mark_ready before ddp_build_buckets");
    new_call(c);
    const int32_t st = mark_one(c, param_id, everyone_mask(c));
    if (st != DDP_OK) return st;
    return flush_or_hold(c);
}

int32_t ddp_mark_ready_local(ddp_ctx* c, int32_t param_id, const uint8_t* used) {
    if (!c) return DDP_ERR_ARG;
    if (!c->built) return fail(c, DDP_ERR_STATE, "ddp_mark_ready_local before ddp_build_buckets");
    if (!used) return fail(c, DDP_ERR_ARG, "ddp_mark_ready_local: used is null");
    new_call(c);
    uint64_t mask = 0;
    for (int32_t r = 0; r < c->R; ++r)
        if (used[r] != 0) mask |= uint64_t(1) << r;
    const int32_t st = mark_one(c, param_id, mask);
    if (st != DDP_OK) return st;
    return flush_or_hold(c);
}

int32_t ddp_mark_ready_many(ddp_ctx* c, const int32_t* ids, int32_t count) {
    if (!c || (count > 0 && !ids) || count < 0) return DDP_ERR_ARG;
    if (!c->built) return fail(c, DDP_ERR_STATE, "ddp_mark_ready_many before ddp_build_buckets");
    new_call(c);
    for (int32_t k = 0; k < count; ++k) {
        const int32_t st = mark_one(c, ids[k], everyone_mask(c));
        if (st != DDP_OK) {
            (void)flush_deferred(c);   // what the earlier marks completed is still launched
            return st;
        }
    }
    return flush_deferred(c);
}

// Stream s waits for what lane l has been given in the running iteration.
static int32_t join_lane(ddp_ctx* c, int l, bool by_flag, hipStream_t s) {
    if (by_flag) {
        const uint64_t tag = static_cast<uint64_t>(c->iteration + 1);
        HIPCHK(c, ddp::launch_done(reinterpret_cast<unsigned long long*>(c->done_word[l]), tag, c->lane[l]));
        HIPCHK(c, hipStreamWaitValue64(s, c->done_word[l], tag, hipStreamWaitValueGte, ~uint64_t(0)));
    } else {
        hipEvent_t ev = l == 0 ? c->ev_done : c->ev_join[l];
        HIPCHK(c, hipEventRecord(ev, c->lane[l]));
        HIPCHK(c, hipStreamWaitEvent(s, ev, 0));
    }
    return DDP_OK;
}

int32_t ddp_finalize_backward(ddp_ctx* c) {
    if (!c) return DDP_ERR_ARG;
    if (!c->built) return fail(c, DDP_ERR_STATE, "ddp_finalize_backward before ddp_build_buckets");
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    const int32_t marks = c->tracker.marks();
    new_call(c);
    std::vector<int32_t> launch;
    c->tracker.drain(launch);
    if (!c->plan_only) HIPCHK(c, hipSetDevice(c->device));
    if (marks < n) {
        // Parameters never marked in this iteration: what earlier no_sync
        // iterations recorded still counts (Section 3.2.4); replicas without any
        // record contribute zeros and are not read.  Every bucket launched
        // before this point was complete, so only the buckets in `launch` can
        // contain such parameters.
        for (int32_t i = 0; i < n; ++i)
            if (!c->tracker.marked(i) && set_participation(c, i, 0)) c->used_running[i] = 1;
    }
    for (int32_t b : launch) note_launch(c, b, marks);
    {
        const int32_t st = flush_deferred(c);
        if (st != DDP_OK) return st;
    }
    if (!c->plan_only) {
        // Every reduction stream that received work joins the backward stream directly.  If the
        // iteration's launches were ordered by device flags, so is the way back: each stream stores the
        // iteration's tag behind its last launch, and the backward stream waits for the value.
        // (Events, recorded there and waited for here behind a kernel that polled for the tags, took the host 10 to
        // 20 us a stream, and the next kernel on the backward stream started 9.4 us after the last one on the
        // reduction stream; it is 4 us of the host and 3.9 us so, however long the wait lasts.)
        const bool by_flag = c->gates_in_iter > 0;
        const unsigned long long tag = static_cast<unsigned long long>(c->iteration + 1);
        // With several streams, and a launch on the backward stream that started as the last of theirs drained, the others' values are
        // waited for on the stream that got the latest launch, and the backward stream waits for that one alone: a wait for a
        // value that is there takes a stream 2.2 us, and that stream has the time.  (ResNet-50, R = 8, one mark per call 160.5 /
        // 158.5 us, with participation masks 128.5 / 126.6; bfloat16, R = 8, 25 MiB buckets 187.5 / 185.2.  Where the backward stream
        // is there first the wait would be on the way: every replica written, R = 3, 25 MiB buckets 73.5 / 75.)
        int last_lane = -1;
        for (int l = 0; l < ddp_ctx::kMaxLanes; ++l)
            if (c->lane_used[l] && c->lane[l] != c->backward && (last_lane < 0 || l == c->latest_lane)) last_lane = l;
        for (int l = 0; l < ddp_ctx::kMaxLanes; ++l) {
            if (!c->lane_used[l] || c->lane[l] == c->backward || l == last_lane) continue;
            const int32_t rc = join_lane(c, l, by_flag, c->tail_chained ? c->lane[last_lane] : c->backward);
            if (rc != DDP_OK) return rc;
        }
        if (last_lane >= 0) {
            const int32_t rc = join_lane(c, last_lane, by_flag, c->backward);
            if (rc != DDP_OK) return rc;
        }
        // from here on the backward stream is behind every bucket launch of the iteration, and
        // what is left runs on it
        if (c->iter_zero) {
            // The bitmap step of Section 4.2: the host bitmap goes to the device
            // with the launch that ORs it over the replicas, which yields the
            // parameters that somebody used.
            const uint64_t* masks = c->local_cur.data();
            const bool by_value = ddp::masks_fit(c->R, n);
            if (!by_value) {
                const int32_t rc = stage_masks(c, 0, n, &masks);
                if (rc != DDP_OK) return rc;
            }
            HIPCHK(c, ddp::launch_bitmap_or(c->d_local, c->d_global, c->h_global, tag, masks, n, c->R, c->backward));
            if (n > ddp::kMasksByValue) c->masks_in_flight[c->iteration & 1] = tag;     // (of this launch, or of a bucket's)
        }
        const bool staged = c->pipeline == DDP_PIPELINE_STAGED;
        if (c->gates_in_iter > 0) {
            // Gates wait a bounded time.  Launches whose gate gave up did nothing; they are
            // redone now that every gradient exists (normally there is none and the launch
            // ends at once).  With a zero participation flag in the iteration the whole
            // bitmap is on the device by now (copied above).
            const ddp::FlatBuckets flat{staged ? c->slabs : nullptr, staged ? c->slab_stride : 0};
            uint32_t dtypes_seen = 0;
            for (const ddp::BucketInfo& bk : c->plan.buckets) dtypes_seen |= 1u << bk.dtype;
            for (int dt = 0; dt < 3; ++dt)
                if (dtypes_seen & (1u << dt))
                    HIPCHK(c, ddp::launch_repair(dt, c->tables, c->d_order,
                                                 c->gate_row(),
                                                 static_cast<int>(c->plan.buckets.size()),
                                                 static_cast<uint32_t>(c->iteration + 1), c->R,
                                                 c->write_all ? c->R : 1, c->iter_zero ? c->d_local : nullptr,
                                                 c->find_unused != 0, make_scale(c->R), 2 * c->num_cus,
                                                 c->nontemporal != 0, flat, c->backward));
        }
        if (c->open_group != static_cast<size_t>(-1)) {      // closes this iteration's bucket launches
            HIPCHK(c, hipEventRecord(c->timed[c->open_group].stop, c->backward));
            c->open_group = static_cast<size_t>(-1);
        }
        if (staged) {
            size_t slot;
            int32_t rc;
            if ((rc = timed_begin(c, DDP_K_UNPACK, -1, c->backward, &slot)) != DDP_OK) return rc;
            HIPCHK(c, ddp::launch_unpack(c->tables, 0, c->h_tile0[n],
                                         c->slabs + static_cast<int64_t>(c->R) * c->slab_stride,
                                         c->write_all ? c->R : 1, c->iter_zero ? c->d_global : nullptr,
                                         c->find_unused != 0, c->backward));
            if ((rc = timed_end(c, slot, c->backward)) != DDP_OK) return rc;
        }
    }
    c->log_closed.swap(c->log_running);
    c->log_running.clear();
    c->order_closed.swap(c->order_running);
    c->order_running.clear();
    c->used_closed = c->used_running;
    std::fill(c->used_running.begin(), c->used_running.end(), 0);
    // host view of the global bitmap (all ones unless a flag was zero)
    for (int32_t i = 0; i < n; ++i) c->global_closed[i] = c->local_cur[c->plan.params[i].segment] != 0 ? 1 : 0;
    c->global_on_device = c->iter_zero && !c->plan_only;
    std::fill(c->acc_used.begin(), c->acc_used.end(), 0);
    std::fill(c->bucket_zero.begin(), c->bucket_zero.end(), 0);
    c->iter_zero = false;
    for (bool& b : c->lane_used) b = false;
    c->launches_in_iter = 0;
    c->gates_in_iter = 0;
    c->prev_launch_ord = 0;
    c->tail_chained = false;
    c->progress_wait = 0;
    c->early_credit = c->late_looks = c->early_launches = 0;
    ++c->iteration;
    c->tracker.new_iteration();
    return DDP_OK;
}

int32_t ddp_get_global_used(ddp_ctx* c, uint8_t* used) {
    if (!c || !used) return DDP_ERR_ARG;
    if (!c->built) return DDP_ERR_STATE;
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    if (c->global_on_device) {
        // what the bitmap kernel of finalize computed and wrote to host memory
        HIPCHK(c, hipSetDevice(c->device));
        const int32_t rc = await_bitmap(c, static_cast<uint64_t>(c->iteration));      // (the closed iteration's tag)
        if (rc != DDP_OK) return rc;
        for (int32_t i = 0; i < n; ++i) used[i] = c->h_global[c->plan.params[i].segment] & 1;
    } else {
        std::memcpy(used, c->global_closed.data(), static_cast<size_t>(n));
    }
    return DDP_OK;
}

int32_t ddp_synchronize(ddp_ctx* c) {
    if (!c) return DDP_ERR_ARG;
    if (c->plan_only) return fail(c, DDP_ERR_NO_DEVICE, "plan-only context has nothing to wait for");
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize(c->backward));
    for (int l = 1; l < ddp_ctx::kMaxLanes; ++l)
        if (c->lane[l]) HIPCHK(c, hipStreamSynchronize(c->lane[l]));
    HIPCHK(c, hipStreamSynchronize(c->reduce));
    c->safe_iteration = c->iteration;
    return DDP_OK;
}

int32_t ddp_get_launch_log(const ddp_ctx* c, int32_t which, int32_t* bucket_ids,
                           int32_t* after_call, int32_t cap, int32_t* n) {
    if (!c || !n || cap < 0 || (which != 0 && which != 1)) return DDP_ERR_ARG;
    const auto& log = which == 0 ? c->log_running : c->log_closed;
    *n = static_cast<int32_t>(log.size());
    for (int32_t i = 0; i < *n && i < cap; ++i) {
        if (bucket_ids) bucket_ids[i] = log[i].first;
        if (after_call) after_call[i] = log[i].second;
    }
    return DDP_OK;
}

// The table that the next micro-step will use was last used micro_slots calls ago: the device must have read it.
// (A word in pinned memory that the copying kernel writes instead of an event: that costs the stream a packet with a
// signal and the host 4 us a record.)  A bounded look, then the stream is waited for.
static int32_t await_micro_slot(ddp_ctx* c) {
    if (c->micro_ticket < static_cast<unsigned long long>(c->micro_slots)) return DDP_OK;
    const unsigned long long need = c->micro_ticket + 1 - static_cast<unsigned long long>(c->micro_slots);
    const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(100);
    while (__atomic_load_n(c->micro_done(), __ATOMIC_ACQUIRE) < need)
        if (std::chrono::steady_clock::now() >= until) {
            HIPCHK(c, hipStreamSynchronize(c->backward));
            break;
        }
    return DDP_OK;
}

// How a micro-step's pointers reach the device: in the arguments of the launch where they fit, as they are or, where
// every replica's tensors lie alike (views into one buffer per replica, say), as R bases and n distances; else as a table.
enum class MicroForm { kTable, kWords, kRegular };

// Fills `words` (kMicroByValue of them) for the two forms that travel by value, and micro_used.
static MicroForm micro_words(ddp_ctx* c, void* const* micro, uint64_t* words) {
    const int64_t R = c->R, n = static_cast<int64_t>(c->plan.params.size());
    if (R + n > ddp::kMicroByValue) return MicroForm::kTable;
    int64_t first = 0;
    while (first < n && micro[first] == nullptr) ++first;
    bool regular = first < n;
    for (int64_t r = 0; regular && r < R; ++r) {
        void* const* const row = micro + r * n;
        const uintptr_t shift = reinterpret_cast<uintptr_t>(row[first]) - reinterpret_cast<uintptr_t>(micro[first]);
        regular = row[first] != nullptr;
        for (int64_t i = 0; regular && i < n; ++i)
            regular = micro[i] == nullptr ? row[i] == nullptr
                                          : row[i] != nullptr && reinterpret_cast<uintptr_t>(row[i]) == reinterpret_cast<uintptr_t>(micro[i]) + shift;
        words[r] = reinterpret_cast<uintptr_t>(row[first]);
    }
    if (regular) {
        const uint64_t everyone = everyone_mask(c);
        for (int64_t i = 0; i < n; ++i) {
            const int32_t segment = c->plan.params[i].segment;
            words[R + segment] = micro[i] ? reinterpret_cast<uintptr_t>(micro[i]) - reinterpret_cast<uintptr_t>(micro[first]) : ddp::kMicroAbsent;
            c->micro_used[segment] = micro[i] ? everyone : 0;
        }
        return MicroForm::kRegular;
    }
    if (R * n > ddp::kMicroByValue) return MicroForm::kTable;
    for (int64_t i = 0; i < n; ++i) {
        const int32_t segment = c->plan.params[i].segment;
        uint64_t used = 0;
        for (int64_t r = 0; r < R; ++r) {
            void* const p = micro[r * n + i];
            words[segment * R + r] = p ? reinterpret_cast<uintptr_t>(p) : ddp::kMicroAbsent;
            used |= static_cast<uint64_t>(p != nullptr) << r;
        }
        c->micro_used[segment] = used;
    }
    return MicroForm::kWords;
}

// Brings a micro-step's pointers to d_micro, through the next of the pinned tables, and notes micro_used.
static int32_t send_micro_table(ddp_ctx* c, void* const* micro) {
    const int64_t R = c->R, n = static_cast<int64_t>(c->plan.params.size());
    void** const table = c->h_micro + static_cast<int64_t>((c->micro_ticket + 1) % static_cast<unsigned long long>(c->micro_slots)) * c->micro_table;
    {
        const int32_t rcw = await_micro_slot(c);
        if (rcw != DDP_OK) return rcw;
    }
    // a parameter at a time: its row of the table is written in one go (R = 32, 1600 tensors: 82 us of
    // host time a call when every pointer went to a cache line of its own, 44 so)
    for (int64_t i = 0; i < n; ++i) {
        const int32_t segment = c->plan.params[i].segment;
        void** row = table + segment * R;
        uint64_t used = 0;
        for (int64_t r = 0; r < R; ++r) {
            void* const p = micro[r * n + i];
            row[r] = p;
            used |= static_cast<uint64_t>(p != nullptr) << r;
        }
        c->micro_used[segment] = used;
    }
    HIPCHK(c, ddp::launch_pointer_copy(c->d_micro, table, c->micro_table, reinterpret_cast<unsigned*>(c->d_micro + c->micro_table),
                                       c->micro_done(), c->micro_ticket + 1, c->backward));
    ++c->micro_ticket;
    return DDP_OK;
}

int32_t ddp_no_sync_accumulate(ddp_ctx* c, void* const* micro) {
    if (!c) return DDP_ERR_ARG;
    if (!c->built) return fail(c, DDP_ERR_STATE, "ddp_no_sync_accumulate before ddp_build_buckets");
    // Section 3.2.4's no_sync covers whole iterations: once a ready mark has been taken, buckets
    // may already be reducing these very tensors in place on another stream.
    if (c->tracker.marks() != 0 || !c->deferred.empty())
        return fail(c, DDP_ERR_STATE, "ddp_no_sync_accumulate in the middle of a synchronizing iteration");
    if (c->plan_only) return fail(c, DDP_ERR_NO_DEVICE, "plan-only context cannot accumulate");
    if (!micro) return fail(c, DDP_ERR_ARG, "ddp_no_sync_accumulate: null pointer array");
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    const int64_t R = c->R;
    // (one addressing of all replicas' rows at a time: the parameter's size is looked at once)
    for (int32_t i = 0; i < n; ++i) {
        uintptr_t any = 0;
        for (int64_t r = 0; r < R; ++r) any |= reinterpret_cast<uintptr_t>(micro[r * n + i]);
        if ((any & static_cast<uintptr_t>(ddp::elem_size(c->plan.params[i].dtype) - 1)) != 0)
            return fail(c, DDP_ERR_ARG, "ddp_no_sync_accumulate: pointer not aligned to its element size");
    }
    HIPCHK(c, hipSetDevice(c->device));
    uint64_t words[ddp::kMicroByValue];
    const MicroForm form = micro_words(c, micro, words);
    if (form == MicroForm::kTable) {
        const int32_t rct = send_micro_table(c, micro);
        if (rct != DDP_OK) return rct;
    }
    size_t slot;
    int32_t rc;
    const unsigned lds = lds_for_blocks(c, c->acc_blocks_per_cu >= 0 ? c->acc_blocks_per_cu
                                                                      : auto_accumulate_blocks(ddp::accumulate_streams(c->h_tile0[n], c->R), c->wide));
    if ((rc = timed_begin(c, DDP_K_ACCUMULATE, -1, c->backward, &slot)) != DDP_OK) return rc;
    if (form == MicroForm::kTable)
        HIPCHK(c, ddp::launch_accumulate(c->tables, c->h_tile0[n], c->R, c->d_micro, lds, c->backward));
    else
        HIPCHK(c, ddp::launch_accumulate_by_value(c->tables, c->h_tile0[n], c->R, words,
                                                  static_cast<int>(form == MicroForm::kRegular ? R + n : R * n),
                                                  form == MicroForm::kRegular, lds, c->backward));
    if ((rc = timed_end(c, slot, c->backward)) != DDP_OK) return rc;
    for (int32_t i = 0; i < n; ++i) {
        const int32_t segment = c->plan.params[i].segment;
        c->acc_used[segment] |= c->micro_used[segment];
        if (c->micro_used[segment] != 0) c->used_running[i] = 1;
    }
    return DDP_OK;
}

int32_t ddp_get_used_map(const ddp_ctx* c, int32_t which, uint8_t* used) {
    if (!c || !used || (which != 0 && which != 1)) return DDP_ERR_ARG;
    if (!c->built) return DDP_ERR_STATE;
    const auto& m = which == 0 ? c->used_running : c->used_closed;
    std::memcpy(used, m.data(), m.size());
    return DDP_OK;
}

int32_t ddp_synth_backward(ddp_ctx* c, const int32_t* order, int32_t count, const int64_t* delay_ns,
                           void* const* src_ptrs, int32_t mark) {
    if (!c) return DDP_ERR_ARG;
    if (!c->built) return fail(c, DDP_ERR_STATE, "ddp_synth_backward before ddp_build_buckets");
    if (c->plan_only) return fail(c, DDP_ERR_NO_DEVICE, "plan-only context cannot run a backward pass");
    if (count < 0 || (count > 0 && !order)) return fail(c, DDP_ERR_ARG, "ddp_synth_backward: bad order");
    const int32_t n = static_cast<int32_t>(c->plan.params.size());
    const int64_t R = c->R;
    for (int32_t k = 0; k < count; ++k) {
        if (order[k] < 0 || order[k] >= n) return fail(c, DDP_ERR_ARG, "ddp_synth_backward: id out of range");
        if (delay_ns && (delay_ns[k] < 0 || delay_ns[k] > 100000000))
            return fail(c, DDP_ERR_ARG, "ddp_synth_backward: delay outside [0, 100 ms]");
    }
    HIPCHK(c, hipSetDevice(c->device));
    new_call(c);
    void** d_rows = nullptr;
    if (src_ptrs && count > 0) {
        const int64_t need = 2 * R * count;
        if (c->emit_in_flight) HIPCHK(c, hipEventSynchronize(c->ev_emit));
        if (need > c->emit_cap) {
            HIPCHK(c, hipStreamSynchronize(c->backward));
            if (c->d_emit) HIPCHK(c, hipFree(c->d_emit));
            if (c->h_emit) HIPCHK(c, hipHostFree(c->h_emit));
            c->d_emit = nullptr; c->h_emit = nullptr; c->emit_cap = 0;
            HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->d_emit), sizeof(void*) * need));
            HIPCHK(c, hipHostMalloc(reinterpret_cast<void**>(&c->h_emit), sizeof(void*) * need, hipHostMallocDefault));
            c->emit_cap = need;
        }
        for (int32_t k = 0; k < count; ++k)
            for (int64_t r = 0; r < R; ++r) {
                void* src = src_ptrs[r * n + order[k]];
                if (!src && c->plan.params[order[k]].numel > 0)
                    return fail(c, DDP_ERR_ARG, "ddp_synth_backward: null source pointer");
                c->h_emit[2 * R * k + r] = c->grad_ptrs[r * n + order[k]];
                c->h_emit[2 * R * k + R + r] = src;
            }
        HIPCHK(c, hipMemcpyAsync(c->d_emit, c->h_emit, sizeof(void*) * need, hipMemcpyHostToDevice, c->backward));
        HIPCHK(c, hipEventRecord(c->ev_emit, c->backward));
        c->emit_in_flight = true;
        d_rows = c->d_emit;
    }
    for (int32_t k = 0; k < count; ++k) {
        const int32_t p = order[k];
        const int64_t ticks = delay_ns ? delay_ns[k] * c->wall_clock_khz / 1000000 : 0;
        if (ticks > 0 || d_rows) {
            // buckets completed so far go out before more backward work is enqueued
            // (unless a launch hold keeps them back for a few more marks)
            const int32_t stf = flush_or_hold(c);
            if (stf != DDP_OK) return stf;
            new_call(c);
            HIPCHK(c, ddp::launch_emit(ticks, d_rows ? d_rows + 2 * R * k : nullptr, c->R,
                                       c->plan.params[p].numel, ddp::elem_size(c->plan.params[p].dtype),
                                       c->emit_busy_blocks,
                                       reinterpret_cast<float*>(c->d_global + round_up(n, 4)),   // spare tail
                                       c->backward));
        }
        if (mark) {
            const int32_t st = mark_one(c, p, everyone_mask(c));
            if (st != DDP_OK) {
                (void)flush_deferred(c);
                return st;
            }
        }
    }
    // with marks this is a call that delivers many of them: what they completed goes out now
    return mark ? flush_deferred(c) : flush_or_hold(c);
}

int32_t ddp_get_kernel_times(ddp_ctx* c, int32_t kind, float* ms, int32_t* ids, int32_t cap,
                             int32_t* n) {
    if (!c || !n || cap < 0) return DDP_ERR_ARG;
    if (c->plan_only) return fail(c, DDP_ERR_NO_DEVICE, "plan-only context has no kernel times");
    HIPCHK(c, hipSetDevice(c->device));
    int32_t k = 0;
    for (const TimedLaunch& t : c->timed) {
        if (t.kind != kind) continue;
        if (k < cap) {
            float v = 0.f;
            HIPCHK(c, hipEventElapsedTime(&v, t.start, t.stop));
            if (ms) ms[k] = v;
            if (ids) ids[k] = t.bucket;
        }
        ++k;
    }
    *n = k;
    return DDP_OK;
}

}  // extern "C"
