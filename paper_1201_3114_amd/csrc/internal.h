// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <condition_variable>
#include <cstddef>
#include <cstdint>
#include <mutex>
#include <string>

#include "../../include/lorenz_cipher.h"

namespace lz {

// ---- errors -------------------------------------------------------------------
void set_error(const char *msg);
int fail(int code, const char *msg);
int hip_fail(hipError_t e, const char *what);
#define LZ_HIP(call)                                        \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return ::lz::hip_fail(e_, #call); \
    } while (0)

// ---- host key setup (keysetup.cpp) ---------------------------------------------
void sha256(const uint8_t *msg, size_t len, uint8_t out[32]);
int key_setup(const uint8_t *pw, size_t n, const lz_params &prm, lz_key &key);
int check_params(const lz_params &prm);
// n <= 2^32 and at most LZ_MAX_BLOCKS blocks of prm.block_len; *nb (may be NULL) = block count
int check_blocks(const lz_params &prm, uint64_t n, uint64_t *nb);

// ---- device-side descriptors -----------------------------------------------------

// Per-message descriptor of the batched and served paths (device memory).
struct MsgDesc {
    double ap[3];        // a'
    double r0[3];        // r0
    uint8_t mu[3], om[3], k[3], decrypt;
    uint32_t nb;         // blocks (chains) of this message, >= 1
    const uint8_t *in;   // message body in
    uint8_t *out;        // message body out
    uint64_t n;          // body length in bytes
};

// Resumable state of one chain (served path), an exact checkpoint.
struct ChainSlot {
    double r[3];
    double al[3];
    uint8_t mu[3], om[3];
    uint8_t fresh;       // 1: state not yet initialised from the key
    uint8_t pad;
    uint32_t pos;        // bytes of this block already processed
    uint32_t len;        // bytes of this block
    uint32_t req;        // request slot
    uint32_t blk;        // block index within the request
    uint32_t pad2;
};

// A chain's checkpoint between two segments of a segment plan (plain and batched paths).
struct ChainState {
    double r[3];
    double al[3];
    uint8_t mu[3], om[3];
    uint8_t pad[2];
};

// The waves of a launch beyond a multiple of the SIMDs, advanced in rounds (plan_segments).
constexpr uint32_t SEG_MAX = 32;  // segments of a block at most
struct SegPlan {
    uint64_t chain0;             // first chain of the plan
    uint32_t waves;              // its waves (0: no plan)
    uint32_t segs, seg_len;      // segments per block and their bytes
    uint32_t rounds;
    uint32_t off[SEG_MAX + 1];   // tasks before segment s
    ChainState *state;           // a checkpoint per chain of the plan
};
// A message or batch between the chain counts of two layouts, run in rounds of both (plan_mix).
struct MixPlan {
    uint32_t rounds;             // 0: no plan
    int ga, gb;                  // lanes per chain of the two layouts
    uint32_t unit, units;        // chains of a unit, units
    uint32_t a;                  // units in ga lanes each round
    uint32_t la, lb;             // bytes a round in ga and in gb lanes
    ChainState *state;           // a checkpoint per chain
};
// Checkpoints of any plan on this many SIMDs: fewer than two waves per SIMD.
ChainState *alloc_checkpoints(int simds);
constexpr size_t seg_state_bytes(int simds) { return (size_t)simds * 2 * 64 * sizeof(ChainState); }

// The two partial-block chains of a stream update, carried by a plain launch as the
// lanes after its nb whole blocks: the head finishes the pending partial block from
// its checkpoint (its digest joins the tag when it completes the block, else the
// checkpoint is saved back), the tail starts the next partial block and saves its
// checkpoint.  Running them in the same launch keeps them from adding a wave to a
// SIMD that already runs whole-block waves, which would make that SIMD, and so the
// launch, take longer.
struct StreamExtra {
    ChainSlot *head_slot;  // null: no head chain
    const uint8_t *head_in;
    uint8_t *head_out;
    uint32_t head_cnt, head_complete;
    ChainSlot *tail_slot;  // null: no tail chain
    const uint8_t *tail_in;
    uint8_t *tail_out;
    uint32_t tail_cnt;
    uint64_t tail_block;
};

// Per-request record of the served path (device memory).
struct ReqDesc {
    MsgDesc m;
    unsigned long long tag[3];  // XOR accumulator of block digests
    uint32_t remaining;         // chains not yet finished
    int32_t status;
    const uint8_t *stored_tag;  // decrypt: the 24 tag bytes of the input
};

struct KernelShape {
    int m;         // chains per lane
    int wg;        // threads per workgroup
    int tile;      // LDS bytes per chain per refill
    int wps;       // resident waves per SIMD (persistent kernel)
    int g = 1;     // lanes per chain, where the device has room (lanes_per_chain)
    int simds = 0; // SIMDs of the device
};

struct DevInfo {
    int cus;
    int lds_per_wg_max;
};

// Words of pinned host memory that calls on several threads take and give back; a call that finds none waits for one.
struct PinnedWords {
    static constexpr int N = 64;
    uint64_t *mem = nullptr;
    std::mutex mu;
    std::condition_variable freed;
    uint64_t used = 0;  // a bit per word

    uint64_t *take() {
        std::unique_lock<std::mutex> g(mu);
        freed.wait(g, [&] { return used != ~0ull; });
        const int i = __builtin_ctzll(~used);
        used |= 1ull << i;
        return mem + i;
    }
    void give(uint64_t *word) {
        {
            std::lock_guard<std::mutex> g(mu);
            used &= ~(1ull << (word - mem));
        }
        freed.notify_one();
    }
};

constexpr int WAVE_LANES = 64;  // lanes of a gfx950 wavefront
constexpr int CU_SIMDS = 4;     // SIMDs of a compute unit

// Words of the plain path's and the streams' tag accumulator: three tag words, then the word in
// which a launch with several lanes per chain is told whether the device has room for it.
constexpr size_t TAG_WORDS = 3, TAG_WIDE = 3;
int lanes_per_chain(uint64_t chains, int m, uint32_t integ, int simds);
SegPlan plan_segments(uint64_t chains, const uint32_t *lens, uint32_t last, const lz_params &prm, int simds);
MixPlan plan_mix(uint64_t chains, const lz_params &prm, int simds);

// ---- kernel launchers (kernels.hip) --------------------------------------------------
hipError_t launch_fill_u64(unsigned long long *p, size_t n, hipStream_t s);
// Clears the tag accumulator (TAG_WORDS and the word after them) and runs the message, its last waves
// by the segment plan or all of it by the mix plan if there is one.
hipError_t launch_plain(const KernelShape &sh, const lz_key &key, const lz_params &prm, int decrypt,
                        const uint8_t *in, uint8_t *out, uint64_t n, unsigned long long *tag_acc, const SegPlan &plan,
                        const MixPlan &mix, hipStream_t s);
// One stream update: its full whole blocks from in / out at global block index
// block_base, plus x's head and tail chains, in one launch or the rounds of a mix plan.
hipError_t launch_stream_step(const KernelShape &shape, const lz_key &key, const lz_params &prm, int decrypt,
                              const uint8_t *in, uint8_t *out, uint64_t full, uint64_t block_base,
                              const StreamExtra &x, unsigned long long *tag_acc, const MixPlan &mix, hipStream_t s);
hipError_t launch_plain_finalize(int decrypt, const unsigned long long *tag_acc, const uint8_t *stored_tag,
                                 uint8_t *tag_out, int32_t *status, uint8_t *body, uint64_t n,
                                 hipStream_t s);
// Batched persistent kernel.  full_prefix[i] = number of full blocks of messages [0, i);
// tail_msg: messages with a partial (or empty) last block, longest first.
struct BatchDev {
    const MsgDesc *msgs;
    const uint64_t *full_prefix;  // n_msg + 1 entries
    const uint32_t *tail_msg;     // n_tail entries
    uint32_t n_msg;
    uint32_t n_tail;
    uint64_t n_full;              // total full blocks
    unsigned long long *tag_acc;  // 3 per message
    unsigned long long *counter;  // work-queue head, the word after the tags
    unsigned long long *wide;     // claim_kernel's answer (several lanes per chain)
    int32_t *const *status_ref;   // decrypt: device slot holding the address of the per-message statuses
};
// Clears the tags and the counter and runs the batch.
hipError_t launch_batch(const KernelShape &sh, const DevInfo &dev, const lz_params &prm, const BatchDev &b,
                        const SegPlan &plan, const MixPlan &mix, hipStream_t s);
hipError_t launch_batch_finalize(const BatchDev &b, int decrypt, hipStream_t s);
// One-thread kernel: *slot = status (ordered on s before a batch replay that reads the slot).
hipError_t launch_set_status_ref(int32_t **slot, int32_t *status, hipStream_t s);

// Served path: advance the listed chains by up to tick_bytes bytes each.
struct TickDev {
    ChainSlot *slots;
    ReqDesc *reqs;
    const uint32_t *list;         // active chain slot indices
    uint32_t n_list;
    uint32_t tick_bytes;
    uint32_t n_narrow, narrow_bytes;  // a mixed tick (narrow_bytes > 0): the list's first n_narrow run a lane each, by this
    uint32_t *others;             // 0; receives ~ the waves in flight beside the tick
    uint32_t *done_queue;         // request slots completed in this tick
    uint32_t *done_count;
};
hipError_t launch_tick(const KernelShape &sh, const lz_params &prm, const TickDev &t, hipStream_t s);
// Bytes a lane-per-chain chain runs while one of TICK_MIX_LANES lanes runs tick_bytes, or 0: no mixed ticks.
constexpr int TICK_MIX_LANES = 4;
uint32_t tick_narrow_bytes(const lz_params &prm, uint32_t tick_bytes);
// How much faster a tick of n chains gets on when w of them run wide by tick_bytes and the rest by narrow_bytes.
double tick_mix_gain(const lz_params &prm, uint32_t tick_bytes, uint32_t narrow_bytes, uint64_t n, uint64_t w);
hipError_t launch_install(ReqDesc *reqs, ChainSlot *slots, const ReqDesc *staged, const uint32_t *meta,
                          const uint32_t *idx, uint32_t n_new, uint32_t block_len, hipStream_t s);
hipError_t launch_req_zero(const ReqDesc *reqs, const uint32_t *req_ids, uint32_t n, hipStream_t s);

// One piece of a batched device-to-device copy (the serving loop's request inputs and outputs).
struct CopyPiece {
    const uint8_t *src;
    uint8_t *dst;
    uint64_t len;
};
constexpr uint64_t COPY_PIECE_BYTES = 1ull << 20;  // requests are cut into pieces of at most this size
// Appends the pieces of one copy of len bytes (at most COPY_PIECE_BYTES each) to arr[n...].
inline void add_copy_pieces(CopyPiece *arr, uint32_t &n, const void *src, void *dst, uint64_t len) {
    for (uint64_t o = 0; o < len; o += COPY_PIECE_BYTES) {
        CopyPiece &p = arr[n++];
        p.src = static_cast<const uint8_t *>(src) + o;
        p.dst = static_cast<uint8_t *>(dst) + o;
        p.len = len - o < COPY_PIECE_BYTES ? len - o : COPY_PIECE_BYTES;
    }
}
// diagnostics merge buffer: workgroup b of the histogram and of the lag sums adds its partial
// results into copy b mod DIAG_MERGE; the kernel that follows sums and clears them
constexpr int DIAG_MERGE = 8;
constexpr size_t DIAG_MERGE_WORDS = (size_t)DIAG_MERGE * 16386;  // 64-bit: 256 bins, or up to 16385 lags + the byte total, a copy
hipError_t launch_copy_many(const CopyPiece *pieces, uint32_t n, hipStream_t s);
// the same from a table in host memory, passed in the kernels' arguments (no upload, so nothing
// waits for the stream): one launch per COPY_ARG_PIECES pieces
constexpr uint32_t COPY_ARG_PIECES = 144;  // with the implicit arguments, under 4 KB of kernel arguments
hipError_t launch_copy_pieces_host(const CopyPiece *pieces, uint32_t n, hipStream_t s);

// The device's count of waves in flight (those of claimed launches that still have to run among them), once s gets to it.
hipError_t read_waves(uint32_t *waves, hipStream_t s);

// The method's scalar pieces over device arrays (R, Theta, F^steps), for checking.
hipError_t launch_unit_r(const double *alpha, const uint8_t *om, size_t n, uint8_t *out, hipStream_t s);
hipError_t launch_unit_theta(const uint8_t *p, const uint8_t *o3, size_t n, double *out, hipStream_t s);
hipError_t launch_unit_lorenz(const lz_params &prm, double *r, size_t n, uint32_t steps, hipStream_t s);

// Streaming: fold the pending partial block into the tag, then write or check the tag.
hipError_t launch_stream_finish(const ChainSlot *slot, int pending, int empty, const lz_key &key,
                                unsigned long long *tag_acc, int decrypt, uint8_t *tag, int32_t *status,
                                hipStream_t s);

size_t lds_bytes(const KernelShape &sh);
bool shape_valid(const KernelShape &sh, const DevInfo &dev);

}  // namespace lz

// ---- context (runtime.cpp) ----------------------------------------------------------
struct lz_ctx {
    int device;
    lz_params prm;
    lz::KernelShape shape;
    lz::DevInfo dev;
    char arch[64];               // gcnArchName of the device
    double tuned_ms;             // last autotune: time of the winning shape's launch
    unsigned long long *ws_tag;  // plain path tag accumulator (TAG_WORDS + 1)
    lz::ChainState *ws_seg;      // plain path checkpoints between rounds (seg_state_bytes, on first use)
    int32_t *ws_status;          // plain path status (synchronous decrypt)
    int32_t *host_status;        // pinned
    lz::PinnedWords entropy_words;  // one for each lz_entropy_value under way
    hipStream_t last_stream;
    hipEvent_t last_event;
    bool has_last;
    // diagnostics merge buffer (DIAG_MERGE_WORDS and the word of last_workgroup), zero between calls: each call clears it
    unsigned long long *diag_merge;
    // diagnostics workspace (grown on demand) and the event that orders its users
    void *diag_ws;
    size_t diag_ws_bytes;
    hipEvent_t diag_event;
    hipStream_t diag_last;
    bool diag_has_last;
};
