// Internal definitions shared by the engine (duplexkv.hip) and the block table
// (kv_table.cpp): the engine object itself.  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

#include "../../include/duplexkv.h"

namespace dkv {

// Admission marks (host only).
// mark[] holds (epoch << 2) | bits, bits: 1 = named by the out list, 2 = by the in list.
struct Marks {
    std::vector<uint32_t> blk, slot;
    uint32_t epoch = 0;
    void reset(size_t nb, size_t ns) { blk.assign(nb, 0); slot.assign(ns, 0); epoch = 0; }
    void next()
    {
        if (++epoch >= (1u << 30)) {
            std::fill(blk.begin(), blk.end(), 0u);
            std::fill(slot.begin(), slot.end(), 0u);
            epoch = 1;
        }
    }
};

// What un-waited calls still use, for refusing a call that would race with one
// of them.  Work on one stream runs in order; the two streams run side by side
// until something joins them (kv_wait, or a launch that carries both
// directions).  A stamp equal to `epoch` means: used since the last join.
struct Hazards {
    std::vector<uint32_t> blk_read, blk_written, slot_read, slot_written;  // by stream_out / stream_in work
    uint32_t epoch = 1;
    bool any = false;  // something was stamped since the last join
    void reset(size_t nb, size_t ns)
    {
        any = false;
        blk_read.assign(nb, 0); blk_written.assign(nb, 0);
        slot_read.assign(ns, 0); slot_written.assign(ns, 0);
        epoch = 1;
    }
    void join()
    {
        any = false;
        if (++epoch == 0xFFFFFFFFu) reset(blk_read.size(), slot_read.size());
    }
    // out part: reads blocks, writes slots, on stream_out; in part: reads slots,
    // writes blocks, on stream_in.  Ids are in range (admission came first).
    bool races(const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii, const int32_t *is,
               int32_t ni) const
    {
        if (!any) return false;
        for (int32_t k = 0; k < no; k++)
            if (blk_written[(size_t)oi[k]] == epoch || slot_read[(size_t)os[k]] == epoch) return true;
        for (int32_t k = 0; k < ni; k++)
            if (blk_read[(size_t)ii[k]] == epoch || slot_written[(size_t)is[k]] == epoch) return true;
        return false;
    }
    void stamp(const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii, const int32_t *is, int32_t ni)
    {
        any = true;
        for (int32_t k = 0; k < no; k++) { blk_read[(size_t)oi[k]] = epoch; slot_written[(size_t)os[k]] = epoch; }
        for (int32_t k = 0; k < ni; k++) { blk_written[(size_t)ii[k]] = epoch; slot_read[(size_t)is[k]] = epoch; }
    }
};

constexpr int kRing = 8;  // descriptor sets that may be in flight
constexpr int kReadPasses = 256;  // most passes of one kv_reader_start
// Tile counters of the link-bound kernels: one pair per stream (launches on a
// stream run one after the other), each pair in a 256-byte stretch of its own.
constexpr int kClaimStride = 64;

// Whether a call's stores to the pool are left to the L2 (non-temporal), which joins what
// several accesses store into one line, although the launch could write them through:
// rotations of much in pieces (what is contiguous in the pool, bytes) of a line and less, or
// in the segments of a layer-first pool below 1 KiB whose slots do not follow one another (of
// 8-byte vectors below 512 bytes, in any slots).  Written through, each part of a line is a
// write of its own on the link, and there it takes room from the reads of the other
// direction.  A call of less than 8 MiB gains more by not waiting for the L2 at its end, and
// one that moves much more one way than the other has room on the link.
//   us, non-temporal / written through, in runs of consecutive slots after the comma:
//   layer-first, 24 MiB each way: 64-byte segments 1509 / 1680, 1289 / 1378; 128 812 / 893,
//   771 / 850; 208 887 / 917, 778 / 692; 400 763 / 803, 657 / 610; 640 617 / 643, 576 / 566;
//   8-byte vectors: 200 1022 / 1069, 801 / 821; 520 716 / 770
//   16 MiB: 520 464 / 495, 442 / 405; 1040 411 / 413, 397 / 376; 1280 370 / 362; 2048 367 / 358
//   2 MiB: 80 173 / 162; 128 135 / 109; 208 124 / 103; 640 91 / 66; 200 122 / 102
//   24 out with 12 in: 64 1375 / 1458; 128 748 / 773; 208 744 / 744; 520 616 / 603
//   6 out with 24 in: 128 757 / 750.  24 out alone: 128 651 / 631; 208 579 / 548; 200 603 / 554
//   block-first, 16 MiB each way: blocks of 128 bytes 1366 / 1439, of 160 1203 / 1196
// These are of tiles on 128-byte lines.  With tiles on stretches (MoveParams::line_mask) a layer-first pool's
// segments of more than a line are slower this way in scattered slots, too, 8-byte ones from 264 bytes on in any: 24 MiB
// each way 208 817 / 793, 400 670 / 631, 640 575 / 554, 1008 585 / 559, 264 761 / 736, 504 641 / 599, but 200 803 / 846,
// 128 779 / 858.
inline bool leaves_to_l2(int vec, uint64_t piece, bool layer_first, uint64_t block_bytes, const int32_t *out_slots,
                         int64_t n_out, int64_t n_in)
{
    const bool line = piece <= 128;
    if ((line ? 8 : 2) * n_in <= n_out || 2 * n_out < n_in || (uint64_t)n_out * block_bytes < (8ull << 20)) return false;
    if (line || piece >= 1024 || !layer_first) return line;
    if (vec < 16 && piece < 512) return true;
    int64_t next = 0;
    for (int64_t i = 1; i < n_out; i++) next += out_slots[i] == out_slots[i - 1] + 1;
    return 2 * next < n_out;
}

inline bool list_bad(const int32_t *p, int32_t n) { return n < 0 || (n > 0 && !p); }

}  // namespace dkv

struct kv_engine;
namespace dkv {
// Blocks until the transfers enqueued so far are done, without closing the
// interval kv_last_stats() reports (kv_wait does that).  No-op when nothing is
// pending.  Defined with the engine; the block table calls it before it hands
// blocks and slots of a finished request to new owners.
int drain(kv_engine *e);
}  // namespace dkv

struct kv_engine {
    kv_config cfg;
    int device = 0;
    uint64_t seg = 0, block_bytes = 0, cache_bytes = 0, pool_bytes = 0;
    uint32_t n_planes = 0;
    int vec = 1;  // bytes per lane access
    uint8_t *hbm = nullptr;
    uint8_t *pool = nullptr;
    bool own_pool = false;
    hipStream_t s_out = nullptr, s_in = nullptr;
    bool own_streams = false;
    int n_cus = 0;

    // descriptor ring: per set [out_ids | out_slots | in_ids | in_slots]
    int32_t *desc_host = nullptr, *desc_dev = nullptr;
    size_t desc_cap = 0;  // ints per set
    // device: [0..1] counters of stream_out's launches, [kClaimStride..+1] of stream_in's
    unsigned int *claim = nullptr;
    // ring_out[k] / ring_in[k] are recorded after the last work that reads set k
    // on each stream; they double as the end-of-work timestamps for the stats
    hipEvent_t ring_out[dkv::kRing] = {}, ring_in[dkv::kRing] = {};
    bool ring_out_rec[dkv::kRing] = {}, ring_in_rec[dkv::kRing] = {};
    int ring_cur = 0;

    dkv::Marks marks;
    dkv::Hazards hazards;
    std::vector<std::pair<int32_t, int32_t>> sort_tmp;  // (slot, id)

    // stats
    hipEvent_t ev_o0 = nullptr, ev_o1 = nullptr, ev_i0 = nullptr, ev_i1 = nullptr;
    hipEvent_t ev_join = nullptr, ev_join_in = nullptr;  // stream_out waits for stream_in / the reverse
    hipEvent_t b_o0 = nullptr, b_o1 = nullptr, b_i0 = nullptr, b_i1 = nullptr;  // this batch's first start / last end
    // The kernel paths: times left by the launches themselves
    // (pinned host memory, MoveParams::stamps): five arrays of kStamps, for a batch's first
    // launch that carries out work, its first that carries in work (which may be the same
    // one), and later ones that carry only out, only in, and both.
    unsigned long long (*stamps)[2] = nullptr;
    double stamp_ms = 0;                // milliseconds per tick
    bool stamping = false;              // this call's launches leave their times, else events do
    int batch_stamps = -1;              // whether this batch's calls do (-1: not decided yet): one clock for all of them
    bool shapes_through = false;        // every launch shape of this engine writes through to the pool
    int begun[2] = {-1, -1};            // the array of the launch that began this batch's out / in work, -1: not yet
    uint32_t stamp_waves[5] = {};       // stamps to look at in each array; 0: none in this batch
    uint32_t stamp_sides[5] = {};       // what those launches carry: 1 out work, 2 in work
    bool batch_open = false;
    bool out_pending = false, in_pending = false;  // work enqueued since the last kv_wait
    bool in_dirty = false;                         // stream_in holds work stream_out has not joined
    bool out_dirty = false;                        // stream_out holds work stream_in has not joined
    hipEvent_t in_behind = nullptr;                // own streams: what the next work on stream_in has to wait for
    bool in_after_out = false;                     // block table in use: in-only work waits for earlier out work
    int n_tables = 0;                              // block tables attached (kv_destroy refuses while any is)
    // Goes up every time the engine has seen all of its enqueued work finished
    // (kv_wait, kv_query answering KV_OK, dkv::drain): what was enqueued under an
    // earlier value is done.
    uint64_t idle_epoch = 0;
    double t0 = 0;
    kv_stats acc{}, last{};
    int sticky = KV_OK;

    // Layer-wise completion of the kernel paths (cfg.chunk_layers > 0): the last
    // transfer call ran as layer_n_chunks launches of layer_chunk layers each and
    // recorded layer_ev_*[c] behind chunk c.  layer_on_out / layer_on_in say which
    // of the two event lists that call recorded (one launch for both directions
    // records on stream_out only).  layer_chunk == 0: the last call was not chunked.
    std::vector<hipEvent_t> layer_ev_out, layer_ev_in;
    int32_t layer_chunk = 0, layer_n_chunks = 0;
    bool layer_on_out = false, layer_on_in = false;

    // staging for SDMA_STAGED: one buffer per direction, chunk_cap bytes each.
    // A direction's pack / copy / unpack all run in order on that direction's
    // stream, so a buffer is never reused before its last reader is done.
    uint8_t *stage_out = nullptr, *stage_in = nullptr;
    uint64_t chunk_cap = 0;

    // synthetic decode reader
    hipStream_t s_read = nullptr;
    int32_t *read_ids = nullptr;               // device, 2 * n_hbm_blocks ints
    int32_t *read_ids_host = nullptr;          // pinned
    unsigned long long *read_part = nullptr;   // device: one sum per workgroup, then two sets of tile counters
    size_t read_turn = 0;                      // the set that the next pass draws from
    unsigned long long *read_sums = nullptr;   // pinned: per workgroup its sum over all passes and its end, then the begins
    int read_wgs = 0;                          // workgroups of the reader under way
    std::vector<hipEvent_t> read_ev;           // passes + 1 timestamps
    int32_t read_passes = 0;
};
