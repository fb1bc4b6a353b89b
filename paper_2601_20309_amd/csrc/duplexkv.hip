// Host side of the KV rotation engine and its C ABI (see include/duplexkv.h).
//
// Paths (how one call's bytes travel):
//   FUSED        one kv_move_kernel launch carries both directions, each lane
//                alternating an out-vector with an in-vector; zero-copy into /
//                out of the pinned pool.  Default for kv_rotate.
//   ZEROCOPY     the same kernel once per direction on the two streams.
//                Default for kv_swap_out / kv_swap_in.
//   SDMA_STAGED  pack kernel -> HBM staging -> hipMemcpyAsync per contiguous
//                host run (DMA engines), and the mirror, chunk after chunk, each
//                direction in order on its own stream.  Uses no compute units
//                for the link itself.
//   NAIVE        one hipMemcpyAsync per segment, the per-segment baseline of
//                Section 4.3.1 of the paper, kept for the benchmark ladder.
//   DMA_BLOCKS   block-first cache and block-first pool: a block is one
//                contiguous region on both sides, one hipMemcpyAsync per block
//                (the paper's "merged segments"), runs of consecutive pairs merged.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "kv_engine.hpp"
#include "kv_kernels.hpp"


namespace {

using dkv::DirDesc;
using dkv::MoveParams;

double now_ms()
{
    using clk = std::chrono::steady_clock;
    return std::chrono::duration<double, std::milli>(clk::now().time_since_epoch()).count();
}

bool config_ok(const kv_config *c)
{
    if (!c) return false;
    if (c->n_layers <= 0 || c->n_kv_heads <= 0 || c->head_dim <= 0 || c->block_size <= 0 ||
        c->elem_bytes <= 0 || c->n_hbm_blocks <= 0 || c->n_host_slots <= 0)
        return false;
    if (c->host_layout != KV_HOST_BLOCK_FIRST && c->host_layout != KV_HOST_LAYER_FIRST) return false;
    if (c->path < KV_PATH_AUTO || c->path > KV_PATH_DMA_BLOCKS) return false;
    if (c->hbm_layout != KV_HBM_LAYER_FIRST && c->hbm_layout != KV_HBM_BLOCK_FIRST) return false;
    if (c->path == KV_PATH_DMA_BLOCKS &&
        (c->hbm_layout != KV_HBM_BLOCK_FIRST || c->host_layout != KV_HOST_BLOCK_FIRST))
        return false;
    if (c->chunk_layers < 0 || c->max_copy_wgs < 0) return false;
    if (c->vecs_per_lane != 0 && c->vecs_per_lane != 1 && c->vecs_per_lane != 2 && c->vecs_per_lane != 4 &&
        c->vecs_per_lane != 8)
        return false;
    if (c->wg_lanes < 0 || c->wg_lanes > dkv::kMaxThreads || c->wg_lanes % 64 != 0) return false;
    // sizes must stay far inside 64 bits
    const long double cache = 2.0L * c->n_layers * (long double)c->n_hbm_blocks * c->block_size *
                              c->n_kv_heads * c->head_dim * c->elem_bytes;
    const long double pool = 2.0L * c->n_layers * (long double)c->n_host_slots * c->block_size *
                             c->n_kv_heads * c->head_dim * c->elem_bytes;
    return cache < 1e18L && pool < 1e18L;
}

// ---- admission (host only) ------------------------------------------------
using dkv::Marks;
using dkv::kClaimStride;
using dkv::kRing;
using dkv::kReadPasses;
using dkv::list_bad;

bool out_of_range(const int32_t *p, int32_t n, int32_t lim)
{
    uint32_t bad = 0;  // no early end: several ids to an instruction
    for (int32_t i = 0; i < n; i++) bad |= (uint32_t)p[i] >= (uint32_t)lim ? 1u : 0u;
    return bad != 0;
}

// Marks `p` with `bit`; reports a repeat inside this list and a hit on the other list.  (A mark of
// this epoch is at least its first one, and no mark is of a later epoch.)
void mark_list(std::vector<uint32_t> &m, uint32_t epoch, const int32_t *p, int32_t n, uint32_t bit,
               bool &dup, bool &overlap)
{
    const uint32_t first = epoch << 2;
    uint32_t *const marks = m.data();
    uint32_t hits = 0;
    for (int32_t i = 0; i < n; i++) {
        uint32_t &w = marks[(size_t)p[i]];
        hits |= w >= first ? w : 0u;
        w = std::max(w, first) | bit;
    }
    dup = dup || (hits & bit) != 0;
    overlap = overlap || (hits & ~bit & 3u) != 0;
}

int admit(const kv_config *c, Marks &mk, const int32_t *oi, const int32_t *os, int32_t no,
          const int32_t *ii, const int32_t *is, int32_t ni)
{
    if (list_bad(oi, no) || list_bad(os, no) || list_bad(ii, ni) || list_bad(is, ni)) return KV_EINVAL;
    if (out_of_range(oi, no, c->n_hbm_blocks) || out_of_range(ii, ni, c->n_hbm_blocks) ||
        out_of_range(os, no, c->n_host_slots) || out_of_range(is, ni, c->n_host_slots))
        return KV_ERANGE;
    mk.next();
    bool dup = false, overlap = false;
    mark_list(mk.blk, mk.epoch, oi, no, 1u, dup, overlap);
    mark_list(mk.blk, mk.epoch, ii, ni, 2u, dup, overlap);
    mark_list(mk.slot, mk.epoch, os, no, 1u, dup, overlap);
    mark_list(mk.slot, mk.epoch, is, ni, 2u, dup, overlap);
    if (dup) return KV_EDUP;
    if (overlap) return KV_EOVERLAP;
    return KV_OK;
}

}  // namespace


namespace {

#define HIPTRY(e, call)                                                                      \
    do {                                                                                     \
        hipError_t err_ = (call);                                                            \
        if (err_ != hipSuccess) {                                                            \
            fprintf(stderr, "duplexkv: %s failed: %s (%s:%d)\n", #call, hipGetErrorString(err_), \
                    __FILE__, __LINE__);                                                     \
            if (e) (e)->sticky = KV_EHIP;                                                    \
            return KV_EHIP;                                                                  \
        }                                                                                    \
    } while (0)

uint64_t seg_of(const kv_config *c)
{
    return (uint64_t)c->block_size * (uint64_t)c->n_kv_heads * (uint64_t)c->head_dim *
           (uint64_t)c->elem_bytes;
}

int pick_vec(const kv_engine *e)
{
    const uint64_t a = (uint64_t)(uintptr_t)e->hbm | (uint64_t)(uintptr_t)e->pool | e->seg;
    for (int v = 16; v > 1; v >>= 1)
        if ((a & (uint64_t)(v - 1)) == 0) return v;
    return 1;
}

// The four id arrays of a launch (device pointers; a direction that is not
// used, or whose slots are the list indices, passes nullptr).
struct MoveIds {
    const int32_t *out_ids, *out_slots, *in_ids, *in_slots;
    bool on_host = false;  // the pointers are the host's, and the lists few enough to be kernel arguments
};

// A launch's shape: workgroups, lanes per workgroup, vectors per lane per tile;
// short_steps: with no more steps than this, a wave per step; limit_u: the
// vectors per lane by which dir_tiles() counts; through: it has waves enough to write
// through to the pool; even: see grid_of(); fixed_rounds: see run_fixed().
struct LinkShape { int wgs, lanes, u, short_steps, limit_u; bool through, even; uint32_t fixed_rounds; };

template <typename... P, typename... A>
void launch(void (*kernel)(P...), dim3 g, dim3 b, hipStream_t s, hipEvent_t stop, const A &...args)
{
    if (stop) hipExtLaunchKernelGGL(kernel, g, b, 0, s, nullptr, stop, 0, args...);
    else hipLaunchKernelGGL(kernel, g, b, 0, s, args...);
}

// Workgroups of a launch.  Its waves are the workers, and no more of them are launched
// than it has steps.  Where they take fixed shares (run_fixed) that come to several rounds,
// no more than fill the last round as well as the others (even): the launch lasts as many round
// trips over the link as it has rounds, and a round with fewer bytes in it is a shorter one.  Rounds of what
// comes in, that is: where the out list is the longer one, the in list's are not to become more (138 KiB
// out with 83 in, 70 steps, 42 with an in tile: by 69 waves 18.4 us, by 35 19.9).  us a call, before
// and so: both ways 144 KiB 21.8 and 20.2, 224 22.8 and 21.4, 288 24.7 and 22.7, 560 30.9 and 28.9, 1 MiB 39.6
// and 38.7, 1.5 MiB in four chunks 67.0 and 65.0; in, 150 KiB 19.3 and 18.2, 300 21.7 and 20.8; out, 300 KiB
// 20.7 and 20.1.  Not where most comes in and the out tiles ride along, nor for two launches at once: with
// a fifth of the waves gone these fill the link no more (400 KiB in with 133 out 24.6 and 25.5, 800 KiB
// each way by two kernels 41.0 and 41.9).
uint32_t grid_of(const LinkShape &sh, const MoveParams &p, uint32_t &steps)
{
    steps = p.mix_q ? p.in.tiles : std::max(p.out.tiles, p.in.tiles);
    const uint32_t waves_per_wg = (uint32_t)sh.lanes / dkv::kWave, most = (steps + waves_per_wg - 1) / waves_per_wg;
    if (most == 0 || steps <= (uint32_t)sh.short_steps || most <= (uint32_t)sh.wgs) return std::max(1u, most);
    auto rounds = [&](uint32_t tiles, uint32_t wgs) { return ((tiles + waves_per_wg - 1) / waves_per_wg + wgs - 1) / wgs; };
    const uint32_t all = rounds(steps, (uint32_t)sh.wgs);
    if (!sh.even || all > p.fixed_rounds) return (uint32_t)sh.wgs;
    const uint32_t fewer = (most + all - 1) / all;
    return rounds(p.in.tiles, fewer) > rounds(p.in.tiles, (uint32_t)sh.wgs) ? (uint32_t)sh.wgs : fewer;
}

// Whether the waves of a link-bound launch draw steps from its counters.
bool draws(const LinkShape &sh, const MoveParams &p)
{
    uint32_t steps;
    const uint64_t waves = (uint64_t)grid_of(sh, p, steps) * ((uint32_t)sh.lanes / dkv::kWave);
    return steps > p.fixed_rounds * waves;
}

// `stop` (may be nullptr) is recorded by the launch itself.
template <int U, bool LINK>
void launch_move_v(int vec, const LinkShape &sh, hipStream_t s, const MoveParams &p, const MoveIds &d, hipEvent_t stop)
{
    uint32_t steps;
    dim3 g(grid_of(sh, p, steps)), b((unsigned)sh.lanes);
    if constexpr (LINK) {
        if (d.on_host) {
            dkv::IdArgs a;
            int32_t *to = a.v;
            for (auto list : {std::make_pair(d.out_ids, p.out.n), {d.out_slots, p.out.n}, {d.in_ids, p.in.n}, {d.in_slots, p.in.n}})
                to = std::copy(list.first, list.first + list.second, to);
            launch(dkv::kv_move_inline_kernel<dkv::u32x4, U>, g, b, s, stop, p, a);
            return;
        }
    }
#define DKV_LAUNCH(V) launch(dkv::kv_move_kernel<V, U, LINK>, g, b, s, stop, p, d.out_ids, d.out_slots, d.in_ids, d.in_slots)
    switch (vec) {
    case 16: DKV_LAUNCH(dkv::u32x4); break;
    case 8: DKV_LAUNCH(dkv::u32x2); break;
    case 4: DKV_LAUNCH(unsigned int); break;
    case 2: DKV_LAUNCH(unsigned short); break;
    default: DKV_LAUNCH(unsigned char); break;
    }
#undef DKV_LAUNCH
}

// Whether a call's lists go into its launches' arguments.
bool ids_inline(const kv_engine *e, int32_t no, int32_t ni)
{
    return e->vec == 16 && 2 * ((int64_t)no + ni) <= (int64_t)dkv::kInlineIds;
}

// link: the far side is host memory (zero-copy paths); else HBM staging.
void launch_move(const LinkShape &sh, int vec, hipStream_t s, const MoveParams &p, const MoveIds &d, bool link,
                 hipEvent_t stop = nullptr)
{
    if (link) {
        switch (sh.u) {
        case 1: launch_move_v<1, true>(vec, sh, s, p, d, stop); break;
        case 2: launch_move_v<2, true>(vec, sh, s, p, d, stop); break;
        case 4: launch_move_v<4, true>(vec, sh, s, p, d, stop); break;
        default: launch_move_v<8, true>(vec, sh, s, p, d, stop); break;
        }
    } else {
        switch (sh.u) {
        case 1: launch_move_v<1, false>(vec, sh, s, p, d, stop); break;
        case 2: launch_move_v<2, false>(vec, sh, s, p, d, stop); break;
        case 4: launch_move_v<4, false>(vec, sh, s, p, d, stop); break;
        default: launch_move_v<8, false>(vec, sh, s, p, d, stop); break;
        }
    }
}

void hbm_strides(const kv_engine *e, uint64_t &plane_stride, uint64_t &block_stride)
{
    if (e->cfg.hbm_layout == KV_HBM_BLOCK_FIRST) {
        plane_stride = e->seg;
        block_stride = (uint64_t)e->n_planes * e->seg;
    } else {
        plane_stride = (uint64_t)e->cfg.n_hbm_blocks * e->seg;
        block_stride = e->seg;
    }
}

// Whether stores to the pool can be written through (see store_host).
bool writes_through(const kv_engine *e) { return e->vec >= 8; }

// What a launch moves to or from the pool at one place of it.
uint64_t piece_bytes(const kv_engine *e)
{
    if (e->cfg.host_layout == KV_HOST_LAYER_FIRST) return e->seg;
    return e->cfg.chunk_layers > 0 ? std::min(e->block_bytes, 2 * (uint64_t)e->cfg.chunk_layers * e->seg) : e->block_bytes;
}

bool leaves_to_l2(const kv_engine *e, const int32_t *out_slots, int32_t no, int32_t ni)
{
    return dkv::leaves_to_l2(e->vec, piece_bytes(e), e->cfg.host_layout == KV_HOST_LAYER_FIRST, e->block_bytes, out_slots, no, ni);
}

bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &c) == hipSuccess) return c != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// Decides whether the launches of this call leave their times.  Events are for what they
// cannot tell: stores that the L2 still holds as a launch's waves end, and launches that are
// recorded into a graph.  (On the caller's streams, too, events are no better: beside work on
// the other one, 2 MiB in took 21 us by them, which no link does.)  held: the call had better
// leave its stores to the L2.  Returns whether they have to be written through nevertheless:
// where calls before it in the batch left their times.
bool decide_stamps(kv_engine *e, bool held)
{
    if (e->batch_stamps < 0) e->batch_stamps = writes_through(e) && e->shapes_through && !held ? 1 : 0;
    e->stamping = e->batch_stamps && (e->own_streams || !(capturing(e->s_out) || capturing(e->s_in)));
    return e->batch_stamps != 0;
}

// Fills the fields common to every launch (`through` is left at 0).
MoveParams base_params(const kv_engine *e)
{
    MoveParams p{};
    p.hbm = e->hbm;
    hbm_strides(e, p.hbm_plane_stride, p.hbm_block_stride);
    p.plane_skip = p.hbm_plane_stride - e->seg;
    p.plane0 = 0;
    p.n_planes = e->n_planes;
    p.vec_per_seg = (uint32_t)(e->seg / (uint64_t)e->vec);
    return p;
}

// Vectors of one group (see MoveParams) over `planes` planes.  Segments that are
// whole tiles are groups by themselves; others are joined to the whole entry where
// the far side holds it in one piece.
uint64_t group_vecs(uint64_t vec_per_seg, uint32_t planes, bool plane_major, bool whole)
{
    const uint64_t entry = vec_per_seg * planes;
    return whole || plane_major || entry >= 0x7FFFFFFFull ? vec_per_seg : entry;
}

// What every piece of the pool that a launch's groups are begins on a multiple of, at most
// kStretch: segments of a layer-first pool, `planes` planes of a block elsewhere.
uint32_t piece_align(const kv_engine *e, uint32_t planes)
{
    const uint64_t piece = e->cfg.host_layout == KV_HOST_LAYER_FIRST ? e->seg : (planes * e->seg) | e->block_bytes;
    const uint64_t a = (uintptr_t)e->pool | piece | dkv::kStretch;
    return (uint32_t)(a & (0 - a));
}

// Whether tiles are moved to begin where a write on the link does (MoveParams::line_mask).
// Vectors of 4 bytes and less are taken as they lie: a line is half an access of theirs or more.
bool inside_lines(int vec, uint32_t align) { return vec >= 8 && align < dkv::kStretch; }

// MoveParams::line_mask for groups of that many vectors in tiles of `tile`.  For vectors of 8 bytes,
// of which a stretch is half an access, lines of 128 bytes do where whole stretches would take
// one more tile.  (840-byte segments in a layer-first pool, 2 MiB / 20 MiB out, in, both ways, us:
// by lines 41, 44, 51 / 392, 420, 469, by stretches 44, 50, 56 / 392, 426, 469; 360 bytes, 20 MiB
// both ways 532 and 554.  16-byte vectors gain nevertheless: 896 bytes, 24 MiB out 464 and 449.)
uint32_t line_mask(int vec, uint32_t align, uint64_t group, uint32_t tile)
{
    if (!inside_lines(vec, align)) return 0;
    auto mask = [&](uint32_t bytes) { return align >= bytes ? 0u : bytes / (uint32_t)vec - 1u; };
    auto tiles = [&](uint32_t m) { return (group + m + tile - 1) / tile; };
    const uint32_t stretch = mask(dkv::kStretch), line = mask(128);
    return vec == 8 && tiles(stretch) > tiles(line) ? line : stretch;
}

// Cuts the planes [plane0, plane0 + n_planes) of every entry into tiles of `u` vectors per
// lane; align: what groups begin on multiples of on the far side; out: the launch writes there.
// Segments that are whole tiles but begin inside stretches are then cut like others: taken as
// they lie, every access would begin and end in a part of one, and each part, written
// through, is a write of its own on the link.  (24 MiB both ways / out, us, taken as they lie and so, in a pool 128
// bytes behind a stretch: layer-first segments of 1 KiB 575 / 498 and 555 / 471, 2 KiB 555 / 493 and 535 / 465, 4 KiB 553 /
// 487 and 528 / 459; 8-byte vectors, whose tiles then have no lines to begin on but may be wider ones, 512 bytes 605 / 476
// and 605 / 476, 2 KiB 540 / 455 and 532 / 455.  16 bytes behind a line: 1 KiB 574 / 472 and 574 / 472, 2 KiB 621 / 470
// and 546 / 466; 64 MiB, 32 KiB segments 1667 / 1216 and 1340 / 1190, by lines.)
void cut_tiles(MoveParams &p, int vec, int u, uint32_t align, bool out)
{
    const bool whole = p.vec_per_seg % ((uint32_t)dkv::kWave * (uint32_t)u) == 0 && !(out && inside_lines(vec, align));
    const uint32_t tile = (uint32_t)dkv::kWave * (uint32_t)(whole ? u : std::min(u, dkv::kMaxRaggedU));
    p.group_vecs = (uint32_t)group_vecs(p.vec_per_seg, p.n_planes, p.plane_major != 0, whole);
    p.groups_per_entry = p.group_vecs == p.vec_per_seg ? p.n_planes : 1u;
    p.line_mask = whole ? 0 : line_mask(vec, align, p.group_vecs, tile);
    p.by_tiles = dkv::make_div((p.group_vecs + p.line_mask + tile - 1) / tile);
    p.by_seg = p.groups_per_entry == 1 ? dkv::make_div(p.vec_per_seg) : dkv::Div{1, 0, 0};
    p.full_tiles = whole ? 1u : 0u;
}

void pool_strides(const kv_engine *e, uint64_t &slot_stride, uint64_t &plane_stride)
{
    if (e->cfg.host_layout == KV_HOST_BLOCK_FIRST) {
        slot_stride = (uint64_t)e->n_planes * e->seg;
        plane_stride = e->seg;
    } else {
        slot_stride = e->seg;
        plane_stride = (uint64_t)e->cfg.n_host_slots * e->seg;
    }
}

// tiles of one direction over `planes` planes; false if the count leaves no
// headroom in 32 bits (the kernels step a tile index by the grid size)
bool dir_tiles(uint32_t n, uint32_t planes, uint32_t tiles_per_seg, uint32_t &tiles)
{
    const uint64_t t = (uint64_t)n * planes * tiles_per_seg;
    if (t >= 0x7FFFFFFFull) return false;
    tiles = (uint32_t)t;
    return true;
}

// The same for a launch whose tiles are cut; the limit is that of tiles of
// `limit_u` vectors per lane, each within a segment.
bool dir_tiles(const MoveParams &p, uint32_t n, int limit_u, uint32_t &tiles)
{
    const uint32_t tile = (uint32_t)dkv::kWave * (uint32_t)limit_u;
    return dir_tiles(n, p.n_planes, (p.vec_per_seg + tile - 1) / tile, tiles) &&
           dir_tiles(n, p.groups_per_entry, p.by_tiles.d, tiles);
}

// One direction's list of n entries, its tiles counted; false if they are too many.
bool fill_dir(const MoveParams &p, uint32_t n, uint32_t iota, int limit_u, DirDesc &d)
{
    d = DirDesc{n, 0, iota, dkv::make_div(std::max(1u, p.plane_major ? n : p.groups_per_entry))};
    return dir_tiles(p, n, limit_u, d.tiles);
}

int acquire_ring(kv_engine *e, int &k)
{
    k = e->ring_cur;
    e->ring_cur = (e->ring_cur + 1) % kRing;
    // set still referenced by enqueued work: let it drain
    if (e->ring_out_rec[k]) HIPTRY(e, hipEventSynchronize(e->ring_out[k]));
    if (e->ring_in_rec[k]) HIPTRY(e, hipEventSynchronize(e->ring_in[k]));
    e->ring_out_rec[k] = e->ring_in_rec[k] = false;
    if (e->in_behind == e->ring_out[k]) e->in_behind = nullptr;  // waited for just now
    return KV_OK;
}

void open_batch(kv_engine *e)
{
    if (!e->batch_open) {
        e->batch_open = true;
        e->b_o0 = e->b_o1 = e->b_i0 = e->b_i1 = nullptr;
        e->begun[0] = e->begun[1] = e->batch_stamps = -1;
        std::fill_n(e->stamp_waves, 5, 0u);
        e->t0 = now_ms();
        e->acc = kv_stats{};
    }
}

// First work of a direction in this batch: timestamp its start on stream s.
int mark_start(kv_engine *e, bool out_side, hipStream_t s)
{
    if (out_side && !e->b_o0) {
        HIPTRY(e, hipEventRecord(e->ev_o0, s));
        e->b_o0 = e->ev_o0;
    }
    if (!out_side && !e->b_i0) {
        HIPTRY(e, hipEventRecord(e->ev_i0, s));
        e->b_i0 = e->ev_i0;
    }
    return KV_OK;
}

// Has a launch leave its times, beside those of later ones where it is the first that carries
// a direction in this batch.
void stamp_launch(kv_engine *e, bool out, bool in, bool drain, const LinkShape &sh, MoveParams &p)
{
    const int at = out && e->begun[0] < 0 ? 0 : in && e->begun[1] < 0 ? 1 : out && in ? 4 : in ? 3 : 2;
    if (out && e->begun[0] < 0) e->begun[0] = at;
    if (in && e->begun[1] < 0) e->begun[1] = at;
    p.stamps = reinterpret_cast<dkv::u64x2 *>(e->stamps + at * (size_t)dkv::kStamps);
    p.drain = drain ? 1u : 0u;
    uint32_t steps;
    const uint32_t waves = grid_of(sh, p, steps) * ((uint32_t)sh.lanes / dkv::kWave);
    e->stamp_waves[at] = std::max(e->stamp_waves[at], std::min(dkv::kStamps, waves));
    e->stamp_sides[at] = (out ? 1u : 0u) | (in ? 2u : 0u);
}

// The batch's time for a direction, first begin to last end (0: nothing was carried).  Ends
// of the batch before may lie beside its own: the clock only goes up, so the latest counts.
double stamped_ms(const kv_engine *e, int side)
{
    unsigned long long first = ~0ull, last = 0;
    for (int array = 0; array < 5; array++) {
        if (!(e->stamp_sides[array] >> side & 1u)) continue;
        for (uint32_t w = 0; w < e->stamp_waves[array]; w++) {
            const unsigned long long *t = e->stamps[array * (size_t)dkv::kStamps + w];
            if (array == e->begun[side]) first = std::min(first, t[0]);
            last = std::max(last, t[1]);
        }
    }
    return last > first ? (double)(last - first) * e->stamp_ms : 0.0;
}

// Last work of a direction in this call: releases descriptor set k and is the
// end timestamp so far.
int mark_end(kv_engine *e, bool out_side, int k, hipStream_t s)
{
    if (out_side) {
        HIPTRY(e, hipEventRecord(e->ring_out[k], s));
        e->ring_out_rec[k] = true;
        e->b_o1 = e->ring_out[k];
        e->out_pending = true;
        e->out_dirty = true;
    } else {
        HIPTRY(e, hipEventRecord(e->ring_in[k], s));
        e->ring_in_rec[k] = true;
        e->b_i1 = e->ring_in[k];
        e->in_pending = true;
        e->in_dirty = true;
    }
    return KV_OK;
}

// Launch shape of a link-bound kernel: workgroups, lanes per workgroup, vectors
// per lane per tile.  Waves are the workers, each with one tile (U KiB per
// direction at 16-byte vectors) in flight; workgroups only pack them.  What
// saturates PCIe Gen5 x16 is bytes in flight; what a kernel running beside the
// copy loses grows with the number of copy waves, steeply once the copy issues
// more than the link drains.  So each kind of launch gets the smallest shape
// that holds its rate both alone and beside an HBM-bound reader (measured,
// scattered 2 MiB blocks; GB/s alone over 512 MiB per direction / beside the
// reader over 4 GiB, and what the reader keeps of its 7.0 TB/s):
//  both directions in one launch:
//     U 1:  96 waves  98.7 /  94.0 (6.00)   112 waves 100.9 / 100.4 (5.79)   128 waves 101.5 / 101.3 (5.53)
//     U 2:  48 waves  96.3 /  91.5 (6.12)    64 waves 101.4 / 100.4 (5.86)    80 waves 101.5 / 101.5 (5.54)
//     U 4:  32 waves 100.8 /  99.2 (5.99)    40 waves 101.4 / 100.4 (5.87)    48 waves 100.5 / 100.2 (5.73)
//     U 8:  20 waves  98.3 /  87.2 (6.28)    24 waves 100.7 /  92.9 (6.17)    32 waves  96.4 /  96.9 (5.97)
//    (68 x U 2 beside 64 and 72 on another day: 101.5 / 101.1, 101.4 / 100.5, 101.5 / 101.3)
//  swap-out alone (written through, so the link paces the waves and every shape moves
//  57.1 alone; what differs is the rate beside the reader and what the reader keeps):
//     U 1:  48 waves 51.4 (6.66)   64 waves 57.0 (6.60)   112 waves 57.1 (5.62)
//     U 2:  28 waves 55.5 (6.72)   36 waves 57.0 (6.61)    68 waves 56.8 (5.70)
//     U 4:  14 waves 55.6 (6.89)   16 waves 57.0 (6.82)    24 waves 57.1 (6.67)
//     U 8:  12 waves 55.8 (6.90)   14 waves 56.9 (6.82)    16 waves 57.1 (6.76)
//  swap-in alone:
//     U 1:  64 waves 50.5 / 47.7 (5.75)   80 waves 57.6 / 56.2 (5.64)    96 waves 57.6 / 57.5 (5.41)
//     U 2:  40 waves 57.1 / 55.2 (5.75)   44 waves 57.6 / 57.3 (5.68)    48 waves 57.6 / 57.5 (5.64)
//     U 4:  20 waves 56.2 / 53.3 (5.81)   24 waves 57.6 / 57.3 (5.71)    28 waves 57.6 / 57.5 (5.65)
//     U 8:  14 waves 57.6 / 51.4 (5.92)   16 waves 57.6 / 54.6 (5.82)
//  both directions in one launch with at least twice as much coming in as
//  going out (the usual rotation once eager copies have run): the rate is the
//  swap-in's, and 32 waves x U 4 hold it (out : in in blocks, GB/s summed alone /
//  beside the reader, reader):
//     8 : 2048    68 x 2  57.8 / 57.8 (5.37)    32 x 4  57.8 / 57.8 (5.66)
//  1024 : 2048    68 x 2  86.3 / 86.1 (5.58)    32 x 4  86.1 / 85.5 (5.83)
//  1536 : 2048    68 x 2 100.7 / 100.4 (5.75)   32 x 4 100.1 / 96.1 (5.93)   (not taken: 68 x 2 stays)
// The same waves packed four or sixteen to a workgroup do no better.
// A configured vecs_per_lane is kept (the wave count follows it; 8 are cut to
// kMaxRaggedU for segments that 8 do not divide); max_copy_wgs
// counts workgroups of wg_lanes lanes and set alone keeps 256-lane workgroups; wg_lanes set
// alone keeps the number of waves.  max_copy_wgs limits what a copy takes from a kernel
// beside it, so a rotation's waves then have one vector per lane each, unless vecs_per_lane
// says otherwise: fewer waves are fewer bytes in flight.  (At most 24 / 48 / 64 / 96 one-wave
// workgroups: 34 / 67 / 86 / 100 GB/s alone, 26 / 50 / 64 / 90 beside the reader, which keeps
// 6.6 / 6.2 / 6.05 / 5.7 of 7.0 TB/s; with vectors enough for 128 KiB in flight it kept 5.5
// beside any of them.)  From kFewWaves one-wave workgroups on the default's waves take no
// more than those would (at most 144: 101.5 / 100.7 GB/s and 5.46 TB/s by 68 x U 2, 101.1 /
// 101.0 and 4.87 by 144 x U 1).  A swap-out has eight vectors per lane then.  Workgroups of
// several waves share the ports of a CU, and do best with one vector per lane (alone, 14 x
// 512 lanes 97 GB/s by U 1, 83 by U 2; 7 x 1024 lanes 77 and 50).
//
// A wave that writes through waits for the host's acknowledgement, so a shape that has
// fewer bytes in flight than fill the link moves less that way, and its stores stay
// non-temporal (`through`; GB/s alone, reader beside in TB/s, non-temporal and written
// through): out 8 x U 8 56.9 (6.80) and 52.8 (6.82), 12 x U 8 56.7 (6.34) and 57.0 (6.71), 16 x
// U 2 57.0 and 54.0, 64 x U 1 56.5 (5.56) and 57.0 (6.45), two workgroups of 14 waves 56.7
// and 50.9; both ways 96 x U 1 100.4 and 98.6, 112 x U 1 100.9 and 100.8, 48 x U 2 99.7 and
// 96.3, 64 x U 2 101.0 and 101.2, 32 x U 4 100.3 and 99.7, 40 x U 4 99.9 and 101.3, 20 x 256
// lanes 86.1 and 78.5, 36 x 256 lanes 101.1 and 101.3; in-heavy 24 x U 4 83.2 and 81.6, 32 x
// U 4 86.1 and 86.2.
//
// Segments that no tile divides, or that begin inside lines, are moved in tiles that span
// segments where the pool holds a block in one piece; otherwise tiles end with their
// segment.  The vectors per lane are those above unless they leave more than an eighth of the tiles empty, then
// the most that leave the least empty (segments of 105 vectors fill one tile of 128 as they
// fill two of 64: 40 MiB in 1343 us by 64, 841 by 128).  The waves are as many more as the
// tiles are emptier, so that as many bytes are in flight, and 1.4 times that where an access
// is parted into more requests than its bytes need: vectors narrower than 16 bytes, and
// swap-ins from segments that are no whole tiles or begin inside stretches of 256 bytes (swap-in of
// 40 MiB, us, without and with: 840-byte segments 761 and 744, 180-byte 1374 and 998, 3360-byte 754
// and 740, of 1200 bytes in blocks of 57600 751 and 742).
// Vectors narrower than 16 bytes (odd segments or pointers) also get more of them per lane, and where
// 8-byte ones have one a lane nevertheless, what moves in gets 1.5 times the waves: alone always, both ways
// where groups are several tiles of which no more than a third is empty.  us without and with; in brackets for 20 MiB
// beside a reader over 8 GiB, and the ms that it loses per GiB moved:
//   24 MiB both ways, layer-first segments of 1048 bytes 596 and 564, 1400 599 and 571, 1160 591 and 558 (563, 2.5 and
//     469, 3.5), of 200 bytes in blocks of 3200 619 and 556 (604, 2.9 and 467, 3.1)
//   a third empty and more: 1000 bytes 588 and 591, 2 MiB 70.5 and 72.6; single tiles: 360 bytes 665 and 692, 2 MiB 75.6
//     and 78.1, 392 bytes 653 and 677
//   1 MiB out with 2.4 in: 1048 bytes 75.6 and 76.6, 1400 71.8 and 70.4; 10 with 24: 1048 bytes 524 and 515, 1160 516 and 505
//   24 MiB in: 392 bytes 619 and 600 (588, 5.1 and 512, 8.2), 1160 579 and 501 (572, 4.6 and 437, 5.3), 200 in blocks
//     596 and 467 (586, 5.3 and 423, 4.8); out is the same either way
// Now, with tiles on lines instead of stretches and before all of this and line_mask (on another card), us for 40 MiB
// both ways / out / in: segments of 1200 bytes 854 / 753 / 750 (855 / 754 / 762; 856 / 756 / 744), in a
// layer-first pool 903 / 773 / 825 (921 / 796 / 828; 968 / 830 / 820), of 840 bytes there 974 / 781 / 862 (979 / 783 /
// 866; 1150 / 870 / 1350).  All of this goes by the tiles as they are cut, configured vectors or not: segments of 1000 vectors
// with vecs_per_lane = 8 are cut by 4, and with the waves of 8 moved at 86 / 56 / 44 GB/s
// both ways / out / in, with those of 4 at 99 / 56 / 57.
enum LinkKind { kBoth, kInHeavy, kOutOnly, kInOnly };
// A launch of no more than kShortKib per direction gets a wave per tile: no second round
// trip over the link.  (One-way launches in 4 KiB tiles then have up to 32 waves where the
// table above has 16 and 24, those in 1 KiB tiles up to 128 where it has 64 to 120, for the
// 15 to 20 us that they take.)  (8 + 8 blocks of 16 KiB:
// 64 waves x U 2 24.8 us, 40 waves 25.1, 16 waves 28.1; 8 blocks in: 32 x U 4 20.3, 24 x U 4
// 20.8.  16 + 16 blocks: 128 waves 30.6, the table's 68 28.0.  With a wave per tile up to
// 512 KiB the reader beside lost 10-14 ms per GiB moved instead of 2-4.)
constexpr int kShortKib = 128;
constexpr int kFewWaves = 112;

LinkShape link_shape(const kv_engine *e, LinkKind kind)
{
    const int cw = e->cfg.max_copy_wgs, cl = e->cfg.wg_lanes, cu = e->cfg.vecs_per_lane;
    const uint64_t vec_per_seg = e->seg / (uint64_t)e->vec;
    const bool plane_major = e->cfg.host_layout == KV_HOST_LAYER_FIRST;
    const uint32_t planes = e->cfg.chunk_layers > 0 ? std::min(2u * (uint32_t)e->cfg.chunk_layers, e->n_planes) : e->n_planes;
    const uint32_t align = piece_align(e, planes);
    const int64_t cap = (int64_t)cw * (cl ? cl : dkv::kThreads) / dkv::kWave;  // configured waves
    const bool packed = cl ? cl > dkv::kWave : cw > 0;
    const bool few = kind == kBoth && !cu && (packed || (cw && cap < kFewWaves));
    int u = cu ? cu : kind == kBoth ? (few ? 1 : 2) : kind == kOutOnly && (cw || cl > 512) ? 8 : 4;
    auto divides = [&](int w) { return vec_per_seg % ((uint64_t)dkv::kWave * (uint64_t)w) == 0; };
    const bool inside = kind != kInOnly && inside_lines(e->vec, align);  // see cut_tiles()
    auto whole = [&](int w) { return divides(w) && !inside; };
    auto filled = [&](int w) {
        const uint64_t tile = (uint64_t)dkv::kWave * (uint64_t)w, g = group_vecs(vec_per_seg, planes, plane_major, false);
        return (double)g / (double)((g + line_mask(e->vec, align, g, (uint32_t)tile) + tile - 1) / tile * tile);
    };
    int limit_u = u;
    if (!cu) {
        limit_u = divides(1) ? u : 1;
        while (!divides(limit_u) && limit_u > 1) limit_u >>= 1;
    }
    if (!cu && whole(1)) {  // whole tiles only: the segment must be a multiple of the tile
        u = limit_u;
    } else if (!cu) {
        u = std::min(dkv::kMaxRaggedU, u * 16 / e->vec);
        int best = u;  // an eighth empty at most, else the fullest
        for (int w = u / 2; w >= 1 && filled(best) < 0.875; w /= 2)
            if (filled(w) > filled(best)) best = w;
        u = best;
    }
    // what the waves follow: the vectors tiles are cut by (cut_tiles), in KiB per tile and
    // direction, and the share of a tile that is not padding, on average
    const int cut = whole(u) ? u : std::min(u, dkv::kMaxRaggedU), kib = cut * e->vec / 16;
    const double fill = whole(u) ? 1.0 : filled(cut);
    int waves;
    switch (kind) {
    case kOutOnly: waves = kib >= 8 ? 14 : kib >= 4 ? 16 : kib >= 2 ? 36 : 64; break;
    case kInOnly: waves = kib >= 8 ? 16 : kib >= 4 ? 24 : kib >= 2 ? 44 : 80; break;
    case kInHeavy: waves = kib >= 8 ? 20 : kib >= 4 ? 32 : kib >= 2 ? 64 : 112; break;
    default: waves = kib >= 8 ? 24 : kib >= 4 ? 38 : kib >= 2 ? 68 : 120; break;
    }
    const bool parted = e->vec < 16 || (kind == kInOnly && (align < dkv::kStretch || !whole(u)));
    waves = (int)(waves * std::min(4.0, (parted && fill >= 0.5 ? 1.4 : 1.0) / fill));
    // tiles of 512 bytes: what comes in is half of what the table counts on
    const bool several = group_vecs(vec_per_seg, planes, plane_major, whole(u)) > (uint64_t)dkv::kWave * (uint64_t)cut;
    if (e->vec == 8 && cut == 1 && (kind == kInOnly || (kind != kOutOnly && several && fill >= 2.0 / 3))) waves += waves / 2;
    LinkShape s;
    s.u = u;
    s.limit_u = limit_u;
    s.lanes = cl ? cl : (cw ? dkv::kThreads : dkv::kWave);
    s.wgs = cw && (few || cu || kind != kBoth) ? cw : std::max(1, waves * dkv::kWave / s.lanes);
    if (cw) s.wgs = std::min(s.wgs, cw);
    s.short_steps = cw || cl || cu ? 0 : kShortKib / std::max(1, kib);
    const int64_t all = (int64_t)s.wgs * s.lanes / dkv::kWave, flight = all * std::max(1, kib);
    s.through = true;
    s.even = kind != kInHeavy;
    s.fixed_rounds = kind == kOutOnly || kind == kInOnly ? dkv::kFixedRounds : dkv::kFixedRoundsBoth;
    if (!cw && !cl && !cu) return s;
    if (kind == kOutOnly) s.through = flight >= 64 && all >= 12 && s.wgs >= 4;
    if (kind == kInHeavy) s.through = flight >= 112 && s.wgs >= 4;
    if (kind == kBoth) s.through = flight >= (packed || kib >= 4 ? 144 : 120);
    return s;
}

// HBM-bound pack / unpack launches.  Measured on one 256 MiB chunk of scattered
// 32 KiB segments (bare kernel time, source in no cache): persistent waves that
// loop over 4 KiB tiles, 2048 workgroups, 93 us; one 4 KiB tile per wave (16384
// workgroups) 89 us; one 1 KiB tile per wave and no loop at all (65536
// workgroups of 4 waves, dealt out by the hardware dispatcher) 86 us = 78 % of
// the HBM peak, against 100 us for the runtime's own device copy of that size.
// The general move kernel pays too much per wave for tiles that small, so this
// shape has a kernel of its own (kv_stage_kernel).  A configured max_copy_wgs (a
// copy that has to stay small beside other kernels) keeps that many persistent
// workgroups of the move kernel with 4 KiB tiles.
// ids: of the chunk's blocks, on the device, or (on_host) few enough to be kernel arguments.
template <bool UNPACK>
void launch_stage(int vec, hipStream_t s, const dkv::StageParams &p, const int32_t *ids, bool on_host)
{
    // four waves to a workgroup for the gather, one for the scatter (see kv_stage_kernel)
    const uint32_t waves_per_wg = UNPACK ? 1u : dkv::kThreads / dkv::kWave;
    dim3 g((p.tiles + waves_per_wg - 1) / waves_per_wg), b(waves_per_wg * dkv::kWave);
    dkv::IdArgs a;
    if (on_host) std::copy(ids, ids + p.n, a.v);
#define DKV_STAGE(V)                                                                               \
    if (on_host) hipLaunchKernelGGL((dkv::kv_stage_inline_kernel<V, UNPACK>), g, b, 0, s, p, a);   \
    else hipLaunchKernelGGL((dkv::kv_stage_kernel<V, UNPACK>), g, b, 0, s, p, ids)
    switch (vec) {
    case 16: DKV_STAGE(dkv::u32x4); break;
    case 8: DKV_STAGE(dkv::u32x2); break;
    case 4: DKV_STAGE(unsigned int); break;
    case 2: DKV_STAGE(unsigned short); break;
    default: DKV_STAGE(unsigned char); break;
    }
#undef DKV_STAGE
}

// ---- FUSED / ZEROCOPY -----------------------------------------------------
// One link-bound launch, or, with cfg.chunk_layers set, one launch per chunk of
// that many layers, lowest layers first, each followed by an event in `ev`, so
// that whoever consumes the blocks (the model's layer l, a writer of the pool)
// can start on a layer while the later ones still move.  A chunk is the same
// kernel over planes [p0, p1) of every block of the call.
// On the engine's own streams the launch records the event itself (its completion
// signal): as a packet of its own it costs the stream 2.8 us (20 launches of 20 us:
// 497 us with records behind them, 442 us without or with signals).  The caller's
// streams may be under capture, which knows recorded events only.
int launch_link(kv_engine *e, const LinkShape &sh, hipStream_t s, const MoveParams &whole, const MoveIds &ids,
                std::vector<hipEvent_t> *ev)
{
    const uint32_t per_chunk = ev ? 2u * (uint32_t)e->cfg.chunk_layers : whole.n_planes;
    uint32_t c = 0;
    for (uint32_t p0 = 0; p0 < whole.n_planes; p0 += per_chunk, c++) {
        MoveParams q = whole;
        q.plane0 = p0;
        q.n_planes = std::min(per_chunk, whole.n_planes - p0);
        const uint64_t begins = p0 * e->seg | piece_align(e, q.n_planes);
        cut_tiles(q, e->vec, sh.u, (uint32_t)(begins & (0 - begins)), whole.out.n > 0);
        // fits: the whole call's counts were checked
        if (!fill_dir(q, q.out.n, 0, sh.limit_u, q.out) || !fill_dir(q, q.in.n, 0, sh.limit_u, q.in)) return KV_EUNSUP;
        q.mix_q = whole.mix_q && q.out.tiles ? (((uint64_t)q.out.tiles << 32) + q.in.tiles - 1) / q.in.tiles : 0;
        // of several launches the first begins first and the last ends last
        const bool last = p0 + per_chunk >= whole.n_planes;
        if (e->stamping && (p0 == 0 || last)) stamp_launch(e, q.out.n > 0, q.in.n > 0, last, sh, q);
        launch_move(sh, e->vec, s, q, ids, true, ev && e->own_streams ? (*ev)[c] : nullptr);
        HIPTRY(e, hipGetLastError());
        e->acc.n_launches += 1;
        if (ev && !e->own_streams) HIPTRY(e, hipEventRecord((*ev)[c], s));
    }
    return KV_OK;
}

int run_zero_copy(kv_engine *e, int path, int k, int32_t no, int32_t ni)
{
    int32_t *dh = e->desc_host + (size_t)k * e->desc_cap;
    const bool held = leaves_to_l2(e, dh + no, no, ni), timed = decide_stamps(e, held);
    const bool fused = path == KV_PATH_FUSED && no > 0 && ni > 0;
    auto params = [&](const LinkShape &sh, unsigned int *claim, bool out, bool hold) {
        MoveParams q = base_params(e);
        q.fixed_rounds = sh.fixed_rounds;
        q.through = out && writes_through(e) && (timed || (sh.through && !hold)) ? 1u : 0u;
        q.claim = claim;
        q.far_out = e->pool;
        q.far_in = e->pool;
        pool_strides(e, q.far_slot_stride_out, q.far_plane_stride_out);
        q.far_slot_stride_in = q.far_slot_stride_out;
        q.far_plane_stride_in = q.far_plane_stride_out;
        q.plane_major = e->cfg.host_layout == KV_HOST_LAYER_FIRST ? 1u : 0u;
        cut_tiles(q, e->vec, sh.u, piece_align(e, e->n_planes), out);
        return q;
    };
    // The link-bound kernels fetch ids and slots with scalar loads, for every tile anew.  A call of
    // few blocks has its lists in the launches' arguments; other lists are uploaded first, ~5 us
    // on the launch's stream: read in place from the pinned ring, over the link, they cost a rotation
    // more, by what an entry stands for (us for 460 + 460 blocks in a block-first pool, in place and uploaded:
    // 28800 bytes a block 288 and 256, 128 KiB 665 and 631, 256 KiB 2460 and 2400, 512 KiB 4813 and 4771, 2 MiB
    // 19010 and 18998; swap-ins half of that, swap-outs a tenth; layer by layer a launch visits
    // an entry for its layers only).  Only where the vectors are too narrow for arguments and a call of few
    // blocks moves much at each place the ring is read in place.
    const bool on_host = ids_inline(e, no, ni);
    const bool few = 2 * ((int64_t)no + ni) <= (int64_t)dkv::kInlineIds && piece_bytes(e) >= (256u << 10);
    const bool upload = !on_host && !few;
    int32_t *dd = upload ? e->desc_dev + (size_t)k * e->desc_cap : dh;
    int32_t *d_o = dd, *d_i = dd + 2 * (size_t)no;  // each: [ids | slots]
    auto upload_ids = [&](bool out_part, bool in_part, hipStream_t s) -> int {
        if (!upload) return KV_OK;
        const size_t a = out_part ? 0 : 2 * (size_t)no, b = in_part ? 2 * ((size_t)no + ni) : 2 * (size_t)no;
        HIPTRY(e, hipMemcpyAsync(dd + a, dh + a, (b - a) * sizeof(int32_t), hipMemcpyHostToDevice, s));
        return KV_OK;
    };
    const DirDesc none{};

    if (fused) {
        // one launch on stream_out carries both directions; stream_in is joined
        // before (if it holds work) and after
        const LinkShape sh = link_shape(e, ni >= 2 * (int64_t)no ? kInHeavy : kBoth);
        // What the out list has beyond the in list is a swap-out on its own: from
        // kSplitBytes on it gets the launch shape of one (16 waves x U 4 instead of 68 x U 2:
        // the same rate, and a co-runner keeps 6.8 instead of 5.7 TB/s),
        // right behind the paired part on the same stream.
        constexpr uint64_t kSplitBytes = 64ull << 20;
        const bool layered = e->cfg.chunk_layers > 0;  // layer by layer: the whole out list stays in the one kernel
        const int32_t n_rest =
            !layered && no > ni && (uint64_t)(no - ni) * e->block_bytes >= kSplitBytes ? no - ni : 0;
        const int32_t no_paired = no - n_rest;
        const LinkShape sh_rest = link_shape(e, kOutOnly);
        MoveParams p = params(sh, e->claim, true, held), p_rest = params(sh_rest, e->claim, true, false);
        p_rest.in = none;
        if (!fill_dir(p, (uint32_t)no_paired, 0, sh.limit_u, p.out) || !fill_dir(p, (uint32_t)ni, 0, sh.limit_u, p.in) ||
            !fill_dir(p_rest, (uint32_t)n_rest, 0, sh_rest.limit_u, p_rest.out))
            return KV_EUNSUP;
        // in list longer: spread the out tiles over it instead of pairing 1:1
        if (p.in.tiles > p.out.tiles)
            p.mix_q = (((uint64_t)p.out.tiles << 32) + p.in.tiles - 1) / p.in.tiles;
        if (e->in_dirty || !e->own_streams) {
            HIPTRY(e, hipEventRecord(e->ev_join, e->s_in));
            HIPTRY(e, hipStreamWaitEvent(e->s_out, e->ev_join, 0));
            e->in_dirty = false;
        }
        if (upload_ids(true, true, e->s_out) != KV_OK) return KV_EHIP;
        if (e->stamping) {
            // launch_link's launches leave their times
        } else if (!e->b_o0 && !e->b_i0) {  // one start timestamp serves both directions
            if (mark_start(e, true, e->s_out) != KV_OK) return KV_EHIP;
            e->b_i0 = e->b_o0;
        } else {
            if (mark_start(e, true, e->s_out) != KV_OK) return KV_EHIP;
            if (!e->b_i0) {
                HIPTRY(e, hipEventRecord(e->ev_i0, e->s_out));
                e->b_i0 = e->ev_i0;
            }
        }
        if (launch_link(e, sh, e->s_out, p, MoveIds{d_o, d_o + no, d_i, d_i + ni, on_host},
                        layered ? &e->layer_ev_out : nullptr) != KV_OK)
            return KV_EHIP;
        e->layer_chunk = layered ? e->cfg.chunk_layers : 0;
        e->layer_on_out = layered;
        e->layer_on_in = false;
        if (n_rest > 0) {
            if (e->stamping) stamp_launch(e, true, false, true, sh_rest, p_rest);
            launch_move(sh_rest, e->vec, e->s_out, p_rest,
                        MoveIds{d_o + no_paired, d_o + no + no_paired, nullptr, nullptr, on_host}, true);
            HIPTRY(e, hipGetLastError());
            e->acc.n_launches += 1;
        }
        if (mark_end(e, true, k, e->s_out) != KV_OK) return KV_EHIP;
        e->b_i1 = e->ring_out[k];
        // What is enqueued on stream_in from now on comes after this call.  Nobody but the
        // engine enqueues on a stream of its own, so there the wait can be left until
        // something is (7 us of host time, and of a queue, per call that has no use for it).
        if (e->own_streams) e->in_behind = e->ring_out[k];
        else HIPTRY(e, hipStreamWaitEvent(e->s_in, e->ring_out[k], 0));
        e->out_dirty = false;
        return KV_OK;
    }
    // One kernel per direction, each on its own stream.  When both run at once
    // they only reach the rate of the fused launch if each has at least one
    // workgroup per CU (measured, one-wave workgroups per kernel, U = 1, 512 + 512
    // MiB: 64 -> 68.9, 112 -> 84.9, 160 -> 92.2, 192 -> 95.1, 256 -> 101.1, 288 -> 101.1
    // GB/s; U = 2: 96 -> 91.3; U = 4: 48 -> 89.2).  With at least twice as much coming in as going out
    // the larger share of fewer, wider waves does better: it leaves the reads their rate (out + in MiB, us with
    // 288 x U 1 each and with 96 + 144 x U 2: 32 + 64 1262 and 1189, 16 + 64 1226 and 1189, 4 + 8 182
    // and 171).  A launch of less than kPairBytes is over before the rate counts: it has the shape
    // of one direction (8 + 8 blocks of 16 KiB 23.0 and 20.8, 30 + 30 31.3 and 29.3; 2 + 2 MiB 64.7 and 66.8), also
    // layer by layer, where many follow one another: in chunks of 800 + 800 KiB 16 in 464 and 424, of 937 + 937 80 in 2514
    // and 2256, of 256 + 256 80 in 1179 and 1044, of 64 + 64 80 in 700 and 702.  (Beside a reader 485 and 458, 2514 and 2418,
    // 1190 and 1222, 859 and 861; it loses 10.5 and 2.0, 9.6 and 1.7, 9.1 and 3.5, 8.9 and 8.6 ms per GiB moved.)
    LinkShape sh_out = link_shape(e, kOutOnly), sh_in = link_shape(e, kInOnly);
    constexpr uint64_t kPairBytes = 1ull << 20;
    const uint64_t planes = e->cfg.chunk_layers > 0 ? std::min(2u * (uint32_t)e->cfg.chunk_layers, e->n_planes) : e->n_planes;
    const bool pair = (uint64_t)std::max(no, ni) * planes * e->seg >= kPairBytes;
    if (no > 0 && ni > 0) sh_out.even = sh_in.even = false;
    if (no > 0 && ni > 0 && pair && !e->cfg.max_copy_wgs && !e->cfg.wg_lanes && !e->cfg.vecs_per_lane) {
        const int cus = e->n_cus > 0 ? e->n_cus : 256;
        const bool in_heavy = ni >= 2 * (int64_t)no && e->seg % (2 * dkv::kWave * (uint64_t)e->vec) == 0;
        sh_out.wgs = in_heavy ? 3 * cus / 8 : 9 * cus / 8;
        sh_in.wgs = in_heavy ? 9 * cus / 16 : 9 * cus / 8;
        sh_out.lanes = sh_in.lanes = dkv::kWave;
        sh_out.u = sh_in.u = sh_out.limit_u = sh_in.limit_u = in_heavy ? 2 : 1;
        sh_out.short_steps = sh_in.short_steps = 0;
    }
    const MoveIds ids_out{d_o, d_o + no, nullptr, nullptr, on_host}, ids_in{nullptr, nullptr, d_i, d_i + ni, on_host};
    // launches on stream_out draw from the first pair of counters, those on stream_in from the second
    MoveParams p_out = params(sh_out, e->claim, true, held), p_in = params(sh_in, e->claim + kClaimStride, false, false);
    p_out.in = p_in.out = none;
    if (!fill_dir(p_out, (uint32_t)no, 0, sh_out.limit_u, p_out.out) ||
        !fill_dir(p_in, (uint32_t)ni, 0, sh_in.limit_u, p_in.in))
        return KV_EUNSUP;  // before anything is enqueued
    // Fixed shares beside one another: both launches' waves take them, up to as many rounds as where a
    // launch has the link to itself, or neither's do beyond the rounds of a launch that carries both
    // directions.  Where one side has its shares and the other draws, the one that draws falls behind.  (us, out + in MiB,
    // limits of 8 and 24 for each side by itself: 2.5 + 2.5 77.6 and 75.3, 3 + 3 89.9 and 86.3, 6 + 6 151.5 and
    // 148.6, beside a reader 83.6 and 80.0, 94.9 and 91.2, 156.0 and 152.9; but 4 + 8, out 21 rounds and in 28, 171.8 and 175.7, in
    // segments of 1200 bytes 184 and 192, 7 + 5 165 and 171, 6 + 7 168 and 183.)  Vectors of 8 bytes gain
    // nothing (840-byte segments, 2.3 + 2.3 89 and 94, 2.8 + 1.9 88 and 91), and layer by layer, where a launch of one
    // side meets several of the other, they lose (8 chunks of 3 + 3 MiB 670 and 754, 10 of 3 + 3 in 1680-byte segments
    // 850 and 1110, 4 of 3.5 + 4.5 440 and 558; short chunks in the shapes of one direction gain: 16 of
    // 0.8 + 0.8 458 and 432).  Configured launches keep to the fewer.
    if (no > 0 && ni > 0) {
        auto shares = [&](const LinkShape &sh, const MoveParams &p, uint32_t tiles) {
            const uint64_t waves = (uint64_t)sh.wgs * (uint64_t)(sh.lanes / dkv::kWave);
            return (uint64_t)tiles * planes <= dkv::kFixedRounds * waves * p.n_planes;
        };
        const bool configured = e->cfg.max_copy_wgs || e->cfg.wg_lanes || e->cfg.vecs_per_lane;
        const bool both = e->vec == 16 && !(pair && e->cfg.chunk_layers) && !configured &&
                          shares(sh_out, p_out, p_out.out.tiles) && shares(sh_in, p_in, p_in.in.tiles);
        p_out.fixed_rounds = p_in.fixed_rounds = both ? dkv::kFixedRounds : dkv::kFixedRoundsBoth;
    }
    // The block table promises that no block or slot is overwritten while an
    // earlier transfer still reads it, and none read while an earlier one still
    // writes it.  Its lists are conflict-free within a call but reuse, across
    // calls, what earlier calls vacated; so each direction of a call first waits
    // for what the other stream was given before this call, whether or not the
    // call carries the other direction too (its own two directions still run
    // side by side).
    if (e->in_after_out && no > 0 && e->in_dirty) {
        // a block this copy-out reads may still be being written by an earlier swap-in
        HIPTRY(e, hipEventRecord(e->ev_join, e->s_in));
        HIPTRY(e, hipStreamWaitEvent(e->s_out, e->ev_join, 0));
        e->in_dirty = false;
    }
    if (e->in_after_out && ni > 0 && e->out_dirty) {
        // a block or slot this swap-in overwrites may still be read by an earlier copy-out
        HIPTRY(e, hipEventRecord(e->ev_join_in, e->s_out));
        HIPTRY(e, hipStreamWaitEvent(e->s_in, e->ev_join_in, 0));
        e->out_dirty = false;
    }
    const bool layered = e->cfg.chunk_layers > 0;
    e->layer_chunk = layered ? e->cfg.chunk_layers : 0;
    e->layer_on_out = layered && no > 0;
    e->layer_on_in = layered && ni > 0;
    if (no > 0) {
        if (upload_ids(true, false, e->s_out) != KV_OK) return KV_EHIP;
        if (!e->stamping && mark_start(e, true, e->s_out) != KV_OK) return KV_EHIP;
        if (launch_link(e, sh_out, e->s_out, p_out, ids_out, layered ? &e->layer_ev_out : nullptr) != KV_OK)
            return KV_EHIP;
        if (mark_end(e, true, k, e->s_out) != KV_OK) return KV_EHIP;
    }
    if (ni > 0) {
        if (upload_ids(false, true, e->s_in) != KV_OK) return KV_EHIP;
        if (!e->stamping && mark_start(e, false, e->s_in) != KV_OK) return KV_EHIP;
        if (launch_link(e, sh_in, e->s_in, p_in, ids_in, layered ? &e->layer_ev_in : nullptr) != KV_OK)
            return KV_EHIP;
        if (mark_end(e, false, k, e->s_in) != KV_OK) return KV_EHIP;
    }
    return KV_OK;
}

// ---- NAIVE: one copy per segment -------------------------------------------
int run_naive(kv_engine *e, const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii,
              const int32_t *is, int32_t ni)
{
    uint64_t ss, ps;
    pool_strides(e, ss, ps);
    uint64_t hps, hbs;
    hbm_strides(e, hps, hbs);
    if (no > 0 && mark_start(e, true, e->s_out) != KV_OK) return KV_EHIP;
    if (ni > 0 && mark_start(e, false, e->s_in) != KV_OK) return KV_EHIP;
    const int32_t nmax = std::max(no, ni);
    for (int32_t i = 0; i < nmax; i++) {  // interleave so both streams fill together
        for (uint32_t pl = 0; pl < e->n_planes; pl++) {
            if (i < no) {
                HIPTRY(e, hipMemcpyAsync(e->pool + (uint64_t)os[i] * ss + pl * ps,
                                         e->hbm + pl * hps + (uint64_t)oi[i] * hbs, e->seg,
                                         hipMemcpyDeviceToHost, e->s_out));
            }
            if (i < ni) {
                HIPTRY(e, hipMemcpyAsync(e->hbm + pl * hps + (uint64_t)ii[i] * hbs,
                                         e->pool + (uint64_t)is[i] * ss + pl * ps, e->seg,
                                         hipMemcpyHostToDevice, e->s_in));
            }
        }
    }
    e->acc.n_launches += (int32_t)(((int64_t)no + ni) * e->n_planes);
    if (no > 0) {
        HIPTRY(e, hipEventRecord(e->ev_o1, e->s_out));
        e->b_o1 = e->ev_o1;
        e->out_pending = e->out_dirty = true;
    }
    if (ni > 0) {
        HIPTRY(e, hipEventRecord(e->ev_i1, e->s_in));
        e->b_i1 = e->ev_i1;
        e->in_pending = e->in_dirty = true;
    }
    return KV_OK;
}

// ---- DMA_BLOCKS: one copy per block, both sides block-first -----------------------
int run_dma_blocks(kv_engine *e, const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii,
                   const int32_t *is, int32_t ni)
{
    const uint64_t bb = e->block_bytes;
    if (no > 0 && mark_start(e, true, e->s_out) != KV_OK) return KV_EHIP;
    if (ni > 0 && mark_start(e, false, e->s_in) != KV_OK) return KV_EHIP;
    int32_t a = 0, b = 0, n_copies = 0;
    while (a < no || b < ni) {  // alternate so both streams fill together
        if (a < no) {
            int32_t r = a + 1;  // run in which block ids and slots both advance by one
            while (r < no && oi[r] == oi[r - 1] + 1 && os[r] == os[r - 1] + 1) r++;
            HIPTRY(e, hipMemcpyAsync(e->pool + (uint64_t)os[a] * bb, e->hbm + (uint64_t)oi[a] * bb,
                                     (uint64_t)(r - a) * bb, hipMemcpyDeviceToHost, e->s_out));
            a = r;
            n_copies++;
        }
        if (b < ni) {
            int32_t r = b + 1;
            while (r < ni && ii[r] == ii[r - 1] + 1 && is[r] == is[r - 1] + 1) r++;
            HIPTRY(e, hipMemcpyAsync(e->hbm + (uint64_t)ii[b] * bb, e->pool + (uint64_t)is[b] * bb,
                                     (uint64_t)(r - b) * bb, hipMemcpyHostToDevice, e->s_in));
            b = r;
            n_copies++;
        }
    }
    e->acc.n_launches += n_copies;
    if (no > 0) {
        HIPTRY(e, hipEventRecord(e->ev_o1, e->s_out));
        e->b_o1 = e->ev_o1;
        e->out_pending = e->out_dirty = true;
    }
    if (ni > 0) {
        HIPTRY(e, hipEventRecord(e->ev_i1, e->s_in));
        e->b_i1 = e->ev_i1;
        e->in_pending = e->in_dirty = true;
    }
    return KV_OK;
}

// ---- SDMA_STAGED -----------------------------------------------------------
// A chunk is blocks [j0, j1) of the slot-sorted list x planes [p0, p1).  Its
// staging image mirrors the host layout ([j][plane][seg] for block-first,
// [plane][j][seg] for layer-first) so that every run of consecutive slots is
// one contiguous range on both sides and costs one DMA copy.
struct ChunkPlan {
    uint32_t blocks_per_chunk, planes_per_chunk;
};

int plan_chunks(const kv_engine *e, uint32_t n, ChunkPlan &pl)
{
    const uint64_t cap = e->chunk_cap;
    if (e->cfg.host_layout == KV_HOST_BLOCK_FIRST) {
        uint32_t planes = e->cfg.chunk_layers > 0 ? std::min<uint32_t>(2u * e->cfg.chunk_layers, e->n_planes)
                                                 : e->n_planes;
        while (planes > 2 && (uint64_t)planes * e->seg > cap) planes -= 2;
        if ((uint64_t)planes * e->seg > cap) return KV_EUNSUP;
        pl.planes_per_chunk = planes;
        pl.blocks_per_chunk = (uint32_t)std::min<uint64_t>(n, cap / ((uint64_t)planes * e->seg));
    } else {
        uint32_t blocks = n;
        if (2ull * blocks * e->seg > cap) blocks = (uint32_t)(cap / (2ull * e->seg));
        if (blocks == 0) return KV_EUNSUP;
        uint32_t layers = (uint32_t)std::min<uint64_t>((uint64_t)e->cfg.n_layers,
                                                        cap / (2ull * blocks * e->seg));
        if (e->cfg.chunk_layers > 0) layers = std::min<uint32_t>(layers, (uint32_t)e->cfg.chunk_layers);
        pl.blocks_per_chunk = blocks;
        pl.planes_per_chunk = 2 * std::max(layers, 1u);
    }
    return KV_OK;
}

// Sorts (slot, id) pairs by slot into the descriptor set: ids at dst[0..n), slots at dst[n..2n).
void sorted_desc(kv_engine *e, const int32_t *ids, const int32_t *slots, int32_t n, int32_t *dst)
{
    e->sort_tmp.resize((size_t)n);
    for (int32_t i = 0; i < n; i++) e->sort_tmp[(size_t)i] = {slots[i], ids[i]};
    std::sort(e->sort_tmp.begin(), e->sort_tmp.end());
    for (int32_t i = 0; i < n; i++) {
        dst[i] = e->sort_tmp[(size_t)i].second;
        dst[(size_t)n + i] = e->sort_tmp[(size_t)i].first;
    }
}

// Copies of one chunk between staging and pool.  `to_host` picks the direction.
//
// A copy costs its DMA engine 3-10 us beyond its bytes, so many short rows of equal
// length at equal distances on both sides go as one two-dimensional copy: the planes of
// a run of slots in a layer-first pool, and the blocks of a run when a chunk holds some
// of their planes.  The DMA engines take such a copy whole at every distance (tried up
// to 1.9 GiB; no kernel runs in its place).  But which engine it lands on depends on the
// process's streams, and it can cost 50 us before its first byte, both directions sharing
// an engine; so rows are joined only where that is still less than a copy each.  20 slots
// out, us as 2, 8, 16, 32 and 80 copies each / joined, at best and at worst:
//     8 KiB rows   155, 480, 930, 1800, 4700 / 230-1035, 260-960, 280-1150, 330-1180, 470
//    64 KiB rows   455, 1660, 3310, 6630, 16500 / 275-1325, 414, 604, 980, 2110
//   and 20 + 15 slots both ways: 64 KiB 515, 1760, 3450, 7000, 17200 / 311-1345, 1860,
//   2780-3180, 3070-3560, 3900-4780;  256 KiB 2400, 2480, 4900, 9700, 24500 /
//   1720-1850, 3060-3560, 3630-4370, 5090-6010, 8930-9460.
// Rows of kOwnCopy and more keep a copy each: those run both ways at 45 GB/s and up.  For
// the same reason scattered whole blocks are not joined in pairs, though any two are
// equally spaced: 120 + 96 blocks of 2 MiB took 8965 us in pairs, 5885 one by one.
constexpr uint64_t kOwnCopy = 512ull << 10, kWideRow = 64ull << 10;
constexpr uint32_t kJoinRows = 32, kJoinWideRows = 16;

int chunk_copies(kv_engine *e, bool to_host, uint8_t *stage, const int32_t *sorted_slots, uint32_t j0,
                 uint32_t j1, uint32_t p0, uint32_t p1, hipStream_t s, int32_t &n_copies)
{
    const uint32_t nb = j1 - j0, np = p1 - p0;
    uint64_t ss, ps;
    pool_strides(e, ss, ps);
    auto copy = [&](uint64_t pool_off, uint64_t stage_off, uint64_t bytes) -> hipError_t {
        n_copies++;
        return to_host ? hipMemcpyAsync(e->pool + pool_off, stage + stage_off, bytes, hipMemcpyDeviceToHost, s)
                       : hipMemcpyAsync(stage + stage_off, e->pool + pool_off, bytes, hipMemcpyHostToDevice, s);
    };
    auto copy_rows = [&](uint64_t pool_off, uint64_t pool_pitch, uint64_t stage_off, uint64_t stage_pitch, uint64_t width,
                         uint32_t rows) -> hipError_t {
        const uint64_t odd = ((uint64_t)(uintptr_t)e->pool | pool_off | stage_off | pool_pitch | stage_pitch | width) & 3u;
        if (rows < (width < kWideRow ? kJoinRows : kJoinWideRows) || width >= kOwnCopy || odd || pool_pitch > 0x7FFFFFFFull || stage_pitch > 0x7FFFFFFFull) {
            hipError_t rc = hipSuccess;
            for (uint32_t r = 0; r < rows && rc == hipSuccess; r++)
                rc = copy(pool_off + r * pool_pitch, stage_off + r * stage_pitch, width);
            return rc;
        }
        n_copies++;
        return to_host ? hipMemcpy2DAsync(e->pool + pool_off, pool_pitch, stage + stage_off, stage_pitch, width, rows,
                                          hipMemcpyDeviceToHost, s)
                       : hipMemcpy2DAsync(stage + stage_off, stage_pitch, e->pool + pool_off, pool_pitch, width, rows,
                                          hipMemcpyHostToDevice, s);
    };
    const bool block_first = e->cfg.host_layout == KV_HOST_BLOCK_FIRST, whole = np == e->n_planes;
    const uint64_t row = (uint64_t)np * e->seg;  // block-first: one block's part of the chunk
    uint32_t j = j0;
    while (j < j1) {  // run of consecutive slots [j, r)
        uint32_t r = j + 1;
        while (r < j1 && sorted_slots[r] == sorted_slots[r - 1] + 1) r++;
        const uint64_t slot = (uint64_t)sorted_slots[j];
        if (block_first && whole) {  // the run is one range
            HIPTRY(e, copy(slot * ss, (j - j0) * row, (r - j) * row));
        } else if (block_first) {
            HIPTRY(e, copy_rows(slot * ss + (uint64_t)p0 * ps, ss, (j - j0) * row, row, row, r - j));
        } else {
            HIPTRY(e, copy_rows(slot * ss + (uint64_t)p0 * ps, ps, (uint64_t)(j - j0) * e->seg, (uint64_t)nb * e->seg,
                                (uint64_t)(r - j) * e->seg, np));
        }
        j = r;
    }
    return KV_OK;
}

MoveParams stage_params(const kv_engine *e, uint8_t *stage, uint32_t nb, uint32_t p0, uint32_t np, int u)
{
    MoveParams p = base_params(e);
    p.plane0 = p0;
    p.n_planes = np;
    p.far_out = p.far_in = stage;
    uint64_t ss, ps;
    if (e->cfg.host_layout == KV_HOST_BLOCK_FIRST) {
        ss = (uint64_t)np * e->seg;
        ps = e->seg;
        p.plane_major = 0;
    } else {
        ss = e->seg;
        ps = (uint64_t)nb * e->seg;
        p.plane_major = 1;
    }
    // the kernel adds plane * ps with the absolute plane index: rebase to p0
    p.far_out = p.far_in = stage - (uint64_t)p0 * ps;
    p.far_slot_stride_out = p.far_slot_stride_in = ss;
    p.far_plane_stride_out = p.far_plane_stride_in = ps;
    cut_tiles(p, e->vec, u, dkv::kStretch, true);  // staging is taken as it lies
    return p;
}

// The same chunk for kv_stage_kernel; false if it has too many tiles for a 32-bit index.
bool stage_kernel_params(const kv_engine *e, uint8_t *stage, uint32_t nb, uint32_t p0, uint32_t np,
                         dkv::StageParams &q)
{
    q = dkv::StageParams{};
    q.hbm = e->hbm;
    q.stage = stage;
    hbm_strides(e, q.hbm_plane_stride, q.hbm_block_stride);
    if (e->cfg.host_layout == KV_HOST_BLOCK_FIRST) {
        q.slot_stride = (uint64_t)np * e->seg;
        q.plane_stride = e->seg;
        q.plane_major = 0;
    } else {
        q.slot_stride = e->seg;
        q.plane_stride = (uint64_t)nb * e->seg;
        q.plane_major = 1;
    }
    q.plane0 = p0;
    q.n_planes = np;
    q.n = nb;
    q.vec_per_seg = (uint32_t)(e->seg / (uint64_t)e->vec);
    q.tiles_per_seg = (q.vec_per_seg + dkv::kWave - 1) / dkv::kWave;
    return dir_tiles(nb, np, q.tiles_per_seg, q.tiles);
}

int run_staged(kv_engine *e, int k, const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii,
               const int32_t *is, int32_t ni)
{
    int32_t *dh = e->desc_host + (size_t)k * e->desc_cap;
    int32_t *dd = e->desc_dev + (size_t)k * e->desc_cap;
    int32_t *h_out = dh, *h_in = dh + 2 * (size_t)no;
    int32_t *d_out = dd, *d_in = dd + 2 * (size_t)no;
    constexpr int U = 4;                         // capped launches: persistent waves, 4 KiB tiles
    const int cap_wgs = e->cfg.max_copy_wgs;     // 0: one wave per 1 KiB tile, kv_stage_kernel
    const LinkShape capped{cap_wgs, dkv::kThreads, U, 0, U, false, false, 0};
    ChunkPlan po{}, pi{};
    if (no > 0) {
        int rc = plan_chunks(e, (uint32_t)no, po);
        if (rc != KV_OK) return rc;
        sorted_desc(e, oi, os, no, h_out);
    }
    if (ni > 0) {
        int rc = plan_chunks(e, (uint32_t)ni, pi);
        if (rc != KV_OK) return rc;
        sorted_desc(e, ii, is, ni, h_in);
    }
    // every chunk's tile count must fit the kernels' 32-bit index: checked for the
    // largest chunk of each direction before anything is enqueued
    {
        const uint64_t vec_per_seg = e->seg / (uint64_t)e->vec;
        const uint64_t tile = (uint64_t)dkv::kWave * (cap_wgs > 0 ? U : 1);
        const uint32_t tiles_per_seg = (uint32_t)((vec_per_seg + tile - 1) / tile);
        uint32_t unused;
        if ((no > 0 && !dir_tiles(po.blocks_per_chunk, po.planes_per_chunk, tiles_per_seg, unused)) ||
            (ni > 0 && !dir_tiles(pi.blocks_per_chunk, pi.planes_per_chunk, tiles_per_seg, unused)))
            return KV_EUNSUP;
    }
    // A chunk of few blocks gets their ids as kernel arguments: a copy ahead of the chunks costs each
    // direction a launch, and the first DMA copy of a swap-in, which needs no ids, a wait for it.
    // (us a call with the copies and without: 2 + 1 blocks of 34 KiB 47.9 and 43.1, 2 + 3 of 128 KiB 62.4 and
    // 55.8, 1 + 1 of 4 MiB 130 and 125, of 5 MiB in 160 planes 149 and 144; 120 + 96 of 2 MiB 5861 and 5865.
    // The arguments of its one-wave workgroups make an unpack kernel 0.5 us longer where a chunk is 256 MiB, 93.1 and 92.5
    // in one run, 0.1 at 64 MiB; the copy costs the call more there, too: blocks of 2 MiB in, 16 629.0 and 625.3, 64
    // 2419.6 and 2416.0, 128 4813.9 and 4808.8, 512 19237 and 19234.)
    const bool args_out = cap_wgs == 0 && po.blocks_per_chunk <= dkv::kInlineIds;
    const bool args_in = cap_wgs == 0 && pi.blocks_per_chunk <= dkv::kInlineIds;
    if (no > 0) {
        if (!args_out) HIPTRY(e, hipMemcpyAsync(d_out, h_out, 2 * (size_t)no * sizeof(int32_t), hipMemcpyHostToDevice, e->s_out));
        if (mark_start(e, true, e->s_out) != KV_OK) return KV_EHIP;
    }
    if (ni > 0) {
        if (!args_in) HIPTRY(e, hipMemcpyAsync(d_in, h_in, 2 * (size_t)ni * sizeof(int32_t), hipMemcpyHostToDevice, e->s_in));
        if (mark_start(e, false, e->s_in) != KV_OK) return KV_EHIP;
    }
    // Chunks of the two directions are enqueued alternately so both streams fill
    // together.  out: pack(c) then its copies; in: copies of c then unpack(c).
    struct Cur { uint32_t j0 = 0, p0 = 0; bool done = true; } co, ci;
    co.done = no == 0;
    ci.done = ni == 0;
    int32_t n_ops = 0;
    // Layer by layer for a consumer (kv_stream_wait_layer): possible when a chunk is
    // chunk_layers layers of the whole list, i.e. the staging buffer did not force
    // the list or the chunk to be cut; then chunk c is layers [c * chunk_layers, ...).
    const uint32_t want_planes = 2u * (uint32_t)e->cfg.chunk_layers;
    const bool lay_out = want_planes && no > 0 && po.blocks_per_chunk >= (uint32_t)no &&
                         po.planes_per_chunk == std::min(want_planes, e->n_planes);
    const bool lay_in = want_planes && ni > 0 && pi.blocks_per_chunk >= (uint32_t)ni &&
                        pi.planes_per_chunk == std::min(want_planes, e->n_planes);
    const bool layered = (lay_out || no == 0) && (lay_in || ni == 0);
    e->layer_chunk = layered ? e->cfg.chunk_layers : 0;
    e->layer_on_out = layered && no > 0;
    e->layer_on_in = layered && ni > 0;
    while (!co.done || !ci.done) {
        if (!co.done) {
            const uint32_t j1 = std::min<uint32_t>(co.j0 + po.blocks_per_chunk, (uint32_t)no);
            const uint32_t p1 = std::min<uint32_t>(co.p0 + po.planes_per_chunk, e->n_planes);
            if (cap_wgs > 0) {
                MoveParams p = stage_params(e, e->stage_out, j1 - co.j0, co.p0, p1 - co.p0, U);
                if (!fill_dir(p, j1 - co.j0, 1, U, p.out)) return KV_EUNSUP;
                launch_move(capped, e->vec, e->s_out, p, MoveIds{d_out + co.j0, nullptr, nullptr, nullptr}, false);
            } else {
                dkv::StageParams q;
                if (!stage_kernel_params(e, e->stage_out, j1 - co.j0, co.p0, p1 - co.p0, q)) return KV_EUNSUP;
                launch_stage<false>(e->vec, e->s_out, q, (args_out ? h_out : d_out) + co.j0, args_out);
            }
            HIPTRY(e, hipGetLastError());
            if (chunk_copies(e, true, e->stage_out, h_out + no, co.j0, j1, co.p0, p1, e->s_out, n_ops) != KV_OK)
                return KV_EHIP;
            if (layered) HIPTRY(e, hipEventRecord(e->layer_ev_out[co.p0 / po.planes_per_chunk], e->s_out));
            n_ops++;
            co.p0 = p1;
            if (co.p0 >= e->n_planes) { co.p0 = 0; co.j0 = j1; }
            co.done = co.j0 >= (uint32_t)no;
        }
        if (!ci.done) {
            const uint32_t j1 = std::min<uint32_t>(ci.j0 + pi.blocks_per_chunk, (uint32_t)ni);
            const uint32_t p1 = std::min<uint32_t>(ci.p0 + pi.planes_per_chunk, e->n_planes);
            if (chunk_copies(e, false, e->stage_in, h_in + ni, ci.j0, j1, ci.p0, p1, e->s_in, n_ops) != KV_OK)
                return KV_EHIP;
            if (cap_wgs > 0) {
                MoveParams p = stage_params(e, e->stage_in, j1 - ci.j0, ci.p0, p1 - ci.p0, U);
                if (!fill_dir(p, j1 - ci.j0, 1, U, p.in)) return KV_EUNSUP;
                launch_move(capped, e->vec, e->s_in, p,
                            MoveIds{nullptr, nullptr, d_in + ci.j0, nullptr}, false);
            } else {
                dkv::StageParams q;
                if (!stage_kernel_params(e, e->stage_in, j1 - ci.j0, ci.p0, p1 - ci.p0, q)) return KV_EUNSUP;
                launch_stage<true>(e->vec, e->s_in, q, (args_in ? h_in : d_in) + ci.j0, args_in);
            }
            HIPTRY(e, hipGetLastError());
            if (layered) HIPTRY(e, hipEventRecord(e->layer_ev_in[ci.p0 / pi.planes_per_chunk], e->s_in));
            n_ops++;
            ci.p0 = p1;
            if (ci.p0 >= e->n_planes) { ci.p0 = 0; ci.j0 = j1; }
            ci.done = ci.j0 >= (uint32_t)ni;
        }
    }
    if (no > 0 && mark_end(e, true, k, e->s_out) != KV_OK) return KV_EHIP;
    if (ni > 0 && mark_end(e, false, k, e->s_in) != KV_OK) return KV_EHIP;
    e->acc.n_launches += n_ops;
    return KV_OK;
}

int ensure_staging(kv_engine *e)
{
    if (e->stage_out) return KV_OK;
    // 256 MiB chunks keep the kernel <-> copy hand-overs (tens of microseconds
    // each) under 1 % of a chunk's link time
    uint64_t cap = e->cfg.staging_bytes ? e->cfg.staging_bytes : (256ull << 20);
    cap -= cap % 256;
    if (cap < 2 * e->seg) return KV_EINVAL;
    e->chunk_cap = cap;
    if (hipMalloc((void **)&e->stage_out, cap) != hipSuccess || hipMalloc((void **)&e->stage_in, cap) != hipSuccess) {
        (void)hipGetLastError();
        return KV_ENOMEM;
    }
    return KV_OK;
}

int transfer(kv_engine *e, const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii,
             const int32_t *is, int32_t ni)
{
    if (!e) return KV_EINVAL;
    if (e->sticky != KV_OK) return e->sticky;
    int rc = admit(&e->cfg, e->marks, oi, os, no, ii, is, ni);
    if (rc != KV_OK) return rc;
    if (no == 0 && ni == 0) return KV_OK;
    int path = e->cfg.path;
    if (path == KV_PATH_AUTO) path = (no > 0 && ni > 0) ? KV_PATH_FUSED : KV_PATH_ZEROCOPY;
    // The block table orders its own calls across the two streams; for everyone
    // else a call that would race with un-waited work on the other stream is
    // refused.  One launch for both directions joins the streams instead.
    const bool joins = path == KV_PATH_FUSED && no > 0 && ni > 0;
    if (!e->in_after_out && !joins && e->hazards.races(oi, os, no, ii, is, ni)) return KV_EBUSY;
    if (path == KV_PATH_SDMA_STAGED) {
        rc = ensure_staging(e);
        if (rc != KV_OK) return rc;
    }
    if (ni > 0 && !joins && e->in_behind) {
        HIPTRY(e, hipStreamWaitEvent(e->s_in, e->in_behind, 0));
        e->in_behind = nullptr;
    }
    open_batch(e);
    e->layer_chunk = 0;  // the kernel paths set it again when they run layer by layer
    if (path == KV_PATH_NAIVE) {
        rc = run_naive(e, oi, os, no, ii, is, ni);
    } else if (path == KV_PATH_DMA_BLOCKS) {
        rc = run_dma_blocks(e, oi, os, no, ii, is, ni);
    } else {
        int k;
        rc = acquire_ring(e, k);
        if (rc != KV_OK) return rc;
        int32_t *dh = e->desc_host + (size_t)k * e->desc_cap;
        if (path != KV_PATH_SDMA_STAGED) {
            int32_t *po = dh, *pi = dh + 2 * (size_t)no;
            if (no) {
                memcpy(po, oi, (size_t)no * sizeof(int32_t));
                memcpy(po + no, os, (size_t)no * sizeof(int32_t));
            }
            if (ni) {
                memcpy(pi, ii, (size_t)ni * sizeof(int32_t));
                memcpy(pi + ni, is, (size_t)ni * sizeof(int32_t));
            }
            rc = run_zero_copy(e, path, k, no, ni);
        } else {
            rc = run_staged(e, k, oi, os, no, ii, is, ni);
        }
    }
    if (rc != KV_OK) return rc;
    if (joins) e->hazards.join();
    else e->hazards.stamp(oi, os, no, ii, is, ni);
    e->acc.bytes_out += (uint64_t)no * e->block_bytes;
    e->acc.bytes_in += (uint64_t)ni * e->block_bytes;
    e->acc.path_used = path;
    return KV_OK;
}

void free_engine(kv_engine *e)
{
    if (!e) return;
    auto ev = [](hipEvent_t &x) { if (x) { (void)hipEventDestroy(x); x = nullptr; } };
    for (int k = 0; k < kRing; k++) { ev(e->ring_out[k]); ev(e->ring_in[k]); }
    ev(e->ev_o0); ev(e->ev_o1); ev(e->ev_i0); ev(e->ev_i1); ev(e->ev_join); ev(e->ev_join_in);
    for (hipEvent_t &x : e->layer_ev_out) ev(x);
    for (hipEvent_t &x : e->layer_ev_in) ev(x);
    if (e->stage_out) (void)hipFree(e->stage_out);
    if (e->stage_in) (void)hipFree(e->stage_in);
    if (e->s_read) (void)hipStreamDestroy(e->s_read);
    if (e->read_ids) (void)hipFree(e->read_ids);
    if (e->read_ids_host) (void)hipHostFree(e->read_ids_host);
    if (e->read_part) (void)hipFree(e->read_part);
    if (e->read_sums) (void)hipHostFree(e->read_sums);
    for (hipEvent_t &x : e->read_ev) ev(x);
    if (e->desc_host) (void)hipHostFree(e->desc_host);
    if (e->desc_dev) (void)hipFree(e->desc_dev);
    if (e->claim) (void)hipFree(e->claim);
    if (e->own_pool && e->pool) (void)hipHostFree(e->pool);
    if (e->own_streams) {
        if (e->s_out) (void)hipStreamDestroy(e->s_out);
        if (e->s_in) (void)hipStreamDestroy(e->s_in);
    }
    delete e;
}

// ---- the entry point that allocates nothing --------------------------------
// Everything kv_rotate keeps in memory the engine allocated (the step counters
// of the move kernel and the device copy of the call's four id lists) lives,
// for kv_rotate_static, in one file-scope array of device memory.  Every GPU the
// library runs on holds its own copy of the array, at its own address, until
// the process ends.  Layout: counter pairs, 256 bytes apart, then the id lists as
// [out_ids | out_slots | in_ids | in_slots].
//
// A call finds its counters at zero whatever calls before it did, also if some of
// those overlapped in time, against the rule, and left the pair they shared at other
// values.  Where the lists are uploaded, or the call is being captured (its pair then
// belongs to the recording), a launch before it zeroes pair 0.  Other calls take the
// other pairs in turn, and each zeroes the next one's: a launch saved.
constexpr int kStaticPairs = 8;
constexpr size_t kStaticPairBytes = 256, kStaticIdsOff = kStaticPairs * kStaticPairBytes;
constexpr size_t kStaticBytes = kStaticIdsOff + 2 * (size_t)KV_STATIC_MAX_BLOCKS * sizeof(int32_t);
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

// In host code `scratch` is only a handle for the symbol, not a device address;
// the address on the current device comes from hipGetSymbolAddress, once per
// device, and only that pointer is ever handed to a kernel.
constexpr int kStaticMaxDevices = 64;
unsigned char *g_scratch_ptr[kStaticMaxDevices] = {};
int g_static_turn[kStaticMaxDevices] = {};  // of the next call that takes a pair in turn

int static_scratch(unsigned char *&ptr, int &dev)
{
    dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kStaticMaxDevices) {
        (void)hipGetLastError();
        return KV_EHIP;
    }
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess || !p) {
            (void)hipGetLastError();
            fprintf(stderr, "duplexkv: hipGetSymbolAddress(scratch) failed on device %d: %s\n", dev,
                    hipGetErrorString(err));
            return KV_EHIP;
        }
        g_scratch_ptr[dev] = (unsigned char *)p;
    }
    ptr = g_scratch_ptr[dev];
    return KV_OK;
}

// The id lists travel to the scratch array as kernel arguments (copied at
// launch, so the caller's arrays are free again when the call returns, and no
// pinned staging buffer is needed): kIdsPerLaunch ints per launch.  The first
// launch of a call also puts the counter pair to zero.
constexpr uint32_t kIdsPerLaunch = 960;
struct IdChunk {
    int32_t v[kIdsPerLaunch];
};

__global__ __launch_bounds__(256) void kv_ids_kernel(const IdChunk c, int32_t *dst, uint32_t n,
                                                     unsigned int *zero)
{
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) dst[i] = c.v[i];
    if (zero && threadIdx.x < 2) zero[threadIdx.x] = 0u;
}

// Admission without marks of cache size: sorted copies in static host arrays.
int32_t g_sorted[4][KV_STATIC_MAX_BLOCKS];

bool sorted_has_repeat(const int32_t *p, int32_t n)
{
    for (int32_t i = 1; i < n; i++)
        if (p[i] == p[i - 1]) return true;
    return false;
}

bool sorted_share(const int32_t *a, int32_t na, const int32_t *b, int32_t nb)
{
    int32_t i = 0, j = 0;
    while (i < na && j < nb) {
        if (a[i] == b[j]) return true;
        if (a[i] < b[j]) i++;
        else j++;
    }
    return false;
}

int admit_static(const kv_config *c, const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii,
                 const int32_t *is, int32_t ni)
{
    if (list_bad(oi, no) || list_bad(os, no) || list_bad(ii, ni) || list_bad(is, ni)) return KV_EINVAL;
    if ((int64_t)no + ni > KV_STATIC_MAX_BLOCKS) return KV_E2BIG;
    if (out_of_range(oi, no, c->n_hbm_blocks) || out_of_range(ii, ni, c->n_hbm_blocks) ||
        out_of_range(os, no, c->n_host_slots) || out_of_range(is, ni, c->n_host_slots))
        return KV_ERANGE;
    const int32_t *src[4] = {oi, os, ii, is};
    const int32_t len[4] = {no, no, ni, ni};
    bool dup = false;
    for (int k = 0; k < 4; k++) {
        if (len[k]) memcpy(g_sorted[k], src[k], (size_t)len[k] * sizeof(int32_t));
        std::sort(g_sorted[k], g_sorted[k] + len[k]);
        dup = dup || sorted_has_repeat(g_sorted[k], len[k]);
    }
    if (dup) return KV_EDUP;
    if (sorted_share(g_sorted[0], no, g_sorted[2], ni) || sorted_share(g_sorted[1], no, g_sorted[3], ni))
        return KV_EOVERLAP;
    return KV_OK;
}

double median(std::vector<double> v)
{
    std::sort(v.begin(), v.end());
    return v[v.size() / 2];
}

}  // namespace

int dkv::drain(kv_engine *e)
{
    if (!e) return KV_EINVAL;
    if (e->sticky != KV_OK) return e->sticky;
    if (e->out_pending) HIPTRY(e, hipStreamSynchronize(e->s_out));
    if (e->in_pending) HIPTRY(e, hipStreamSynchronize(e->s_in));
    e->idle_epoch++;
    return KV_OK;
}

extern "C" {

uint64_t kv_seg_bytes(const kv_config *c) { return config_ok(c) ? seg_of(c) : 0; }
uint64_t kv_block_bytes(const kv_config *c) { return config_ok(c) ? 2ull * c->n_layers * seg_of(c) : 0; }
uint64_t kv_cache_bytes(const kv_config *c)
{
    return config_ok(c) ? kv_block_bytes(c) * (uint64_t)c->n_hbm_blocks : 0;
}
uint64_t kv_pool_bytes(const kv_config *c)
{
    return config_ok(c) ? kv_block_bytes(c) * (uint64_t)c->n_host_slots : 0;
}

int kv_validate(const kv_config *cfg, const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii,
                const int32_t *is, int32_t ni)
{
    if (!config_ok(cfg)) return KV_EINVAL;
    Marks mk;
    mk.reset((size_t)cfg->n_hbm_blocks, (size_t)cfg->n_host_slots);
    return admit(cfg, mk, oi, os, no, ii, is, ni);
}

int kv_create(kv_engine **out, const kv_config *cfg, void *hbm_cache, void *host_pool, void *stream_out,
              void *stream_in)
{
    if (!out) return KV_EINVAL;
    *out = nullptr;
    if (!config_ok(cfg) || !hbm_cache) return KV_EINVAL;
    if ((stream_out == nullptr) != (stream_in == nullptr)) return KV_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
        (void)hipGetLastError();
        fprintf(stderr, "duplexkv: no HIP device is visible\n");
        return KV_EHIP;
    }
    kv_engine *e = new (std::nothrow) kv_engine;
    if (!e) return KV_ENOMEM;
    e->cfg = *cfg;
    e->seg = seg_of(cfg);
    e->n_planes = 2u * (uint32_t)cfg->n_layers;
    e->block_bytes = kv_block_bytes(cfg);
    e->cache_bytes = kv_cache_bytes(cfg);
    e->pool_bytes = kv_pool_bytes(cfg);
    e->hbm = (uint8_t *)hbm_cache;
    int rc = KV_OK;
    auto fail = [&](int code) { free_engine(e); return code; };

    if (hipGetDevice(&e->device) != hipSuccess) return fail(KV_EHIP);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, e->device) != hipSuccess) return fail(KV_EHIP);
    e->n_cus = prop.multiProcessorCount;

    // the cache pointer must be a device allocation that really spans cache_bytes
    {
        hipDeviceptr_t base = nullptr;
        size_t span = 0;
        if (hipMemGetAddressRange(&base, &span, (hipDeviceptr_t)hbm_cache) != hipSuccess) {
            (void)hipGetLastError();
            fprintf(stderr, "duplexkv: hbm_cache is not a device allocation\n");
            return fail(KV_EINVAL);
        }
        const uintptr_t lo = (uintptr_t)base, hi = lo + span, p = (uintptr_t)hbm_cache;
        if (p < lo || p + e->cache_bytes > hi) {
            fprintf(stderr, "duplexkv: hbm_cache allocation is smaller than the configured cache\n");
            return fail(KV_EINVAL);
        }
    }
    if (host_pool) {
        hipPointerAttribute_t at;
        if (hipPointerGetAttributes(&at, host_pool) != hipSuccess || at.type != hipMemoryTypeHost) {
            (void)hipGetLastError();
            fprintf(stderr, "duplexkv: host_pool is not pinned host memory\n");
            return fail(KV_EINVAL);
        }
        hipDeviceptr_t base = nullptr;
        size_t span = 0;
        if (hipMemGetAddressRange(&base, &span, (hipDeviceptr_t)host_pool) == hipSuccess) {
            const uintptr_t lo = (uintptr_t)base, hi = lo + span, p = (uintptr_t)host_pool;
            if (p < lo || p + e->pool_bytes > hi) {
                fprintf(stderr, "duplexkv: host_pool allocation is smaller than the configured pool\n");
                return fail(KV_EINVAL);
            }
        } else {
            (void)hipGetLastError();
        }
        e->pool = (uint8_t *)host_pool;
    } else {
        if (hipHostMalloc((void **)&e->pool, e->pool_bytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            e->pool = nullptr;
            return fail(KV_ENOMEM);
        }
        e->own_pool = true;
    }
    e->vec = pick_vec(e);
    e->shapes_through = link_shape(e, kBoth).through && link_shape(e, kInHeavy).through && link_shape(e, kOutOnly).through;

    if (stream_out) {
        e->s_out = (hipStream_t)stream_out;
        e->s_in = (hipStream_t)stream_in;
    } else {
        e->own_streams = true;
        if (hipStreamCreateWithFlags(&e->s_out, hipStreamNonBlocking) != hipSuccess ||
            hipStreamCreateWithFlags(&e->s_in, hipStreamNonBlocking) != hipSuccess)
            return fail(KV_EHIP);
    }
    // one call names at most min(blocks, slots) ids over both directions
    e->desc_cap = 2 * (size_t)std::min(cfg->n_hbm_blocks, cfg->n_host_slots) + 16;
    static_assert(kRing * sizeof(int32_t) % sizeof(*e->stamps) == 0);  // the time stamps lie behind the sets
    const size_t sets = kRing * e->desc_cap * sizeof(int32_t), stamps = 5 * (size_t)dkv::kStamps * sizeof(*e->stamps);
    if (hipHostMalloc((void **)&e->desc_host, sets + stamps, hipHostMallocDefault) != hipSuccess ||
        hipMalloc((void **)&e->desc_dev, kRing * e->desc_cap * sizeof(int32_t)) != hipSuccess ||
        hipMalloc((void **)&e->claim, 2 * kClaimStride * sizeof(unsigned int)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(KV_ENOMEM);
    }
    e->stamps = reinterpret_cast<unsigned long long(*)[2]>(e->desc_host + kRing * e->desc_cap);
    memset(e->stamps, 0, stamps);
    int khz = 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, e->device) != hipSuccess || khz <= 0) return fail(KV_EHIP);
    e->stamp_ms = 1.0 / khz;
    // the tile counters start at zero; every launch leaves them at zero again
    if (hipMemset(e->claim, 0, 2 * kClaimStride * sizeof(unsigned int)) != hipSuccess)
        return fail(KV_EHIP);
    bool ok = true;
    for (int k = 0; k < kRing; k++) {
        ok = ok && hipEventCreate(&e->ring_out[k]) == hipSuccess;
        ok = ok && hipEventCreate(&e->ring_in[k]) == hipSuccess;
    }
    for (hipEvent_t *x : {&e->ev_o0, &e->ev_o1, &e->ev_i0, &e->ev_i1}) ok = ok && hipEventCreate(x) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&e->ev_join, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&e->ev_join_in, hipEventDisableTiming) == hipSuccess;
    if (cfg->chunk_layers > 0) {
        e->layer_n_chunks = (cfg->n_layers + cfg->chunk_layers - 1) / cfg->chunk_layers;
        e->layer_ev_out.assign((size_t)e->layer_n_chunks, nullptr);
        e->layer_ev_in.assign((size_t)e->layer_n_chunks, nullptr);
        for (hipEvent_t &x : e->layer_ev_out) ok = ok && hipEventCreateWithFlags(&x, hipEventDisableTiming) == hipSuccess;
        for (hipEvent_t &x : e->layer_ev_in) ok = ok && hipEventCreateWithFlags(&x, hipEventDisableTiming) == hipSuccess;
    }
    if (!ok) return fail(KV_EHIP);
    e->marks.reset((size_t)cfg->n_hbm_blocks, (size_t)cfg->n_host_slots);
    e->hazards.reset((size_t)cfg->n_hbm_blocks, (size_t)cfg->n_host_slots);
    if (cfg->path == KV_PATH_SDMA_STAGED) {
        rc = ensure_staging(e);
        if (rc != KV_OK) return fail(rc);
    }
    *out = e;
    return KV_OK;
}

int kv_destroy(kv_engine *e)
{
    if (!e) return KV_EINVAL;
    if (e->n_tables > 0) return KV_EBUSY;  // a block table still points at this engine
    if (e->s_read) (void)hipStreamSynchronize(e->s_read);
    (void)hipStreamSynchronize(e->s_out);
    (void)hipStreamSynchronize(e->s_in);
    free_engine(e);
    return KV_OK;
}

int kv_swap_out(kv_engine *e, const int32_t *ids, const int32_t *slots, int32_t n)
{
    return transfer(e, ids, slots, n, nullptr, nullptr, 0);
}

int kv_swap_in(kv_engine *e, const int32_t *slots, const int32_t *ids, int32_t n)
{
    return transfer(e, nullptr, nullptr, 0, ids, slots, n);
}

int kv_rotate(kv_engine *e, const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii,
              const int32_t *is, int32_t ni)
{
    return transfer(e, oi, os, no, ii, is, ni);
}

int kv_wait(kv_engine *e)
{
    if (!e) return KV_EINVAL;
    if (e->sticky != KV_OK) return e->sticky;
    // Only streams this engine put work on are waited for.  (Waiting for the event behind
    // the last call instead is 3 us shorter, and leaves the runtime with a stream it has
    // not seen idle: every allocation and device-wide wait of the process pays for that.)
    for (int side = 0; side < 2; side++) {
        const bool pending = side == 0 ? e->out_pending : e->in_pending;
        if (!pending) continue;
        HIPTRY(e, hipStreamSynchronize(side == 0 ? e->s_out : e->s_in));
    }
    e->out_pending = e->in_pending = false;
    e->out_dirty = e->in_dirty = false;
    e->in_behind = nullptr;
    e->hazards.join();
    e->idle_epoch++;
    for (int k = 0; k < kRing; k++) e->ring_out_rec[k] = e->ring_in_rec[k] = false;
    if (e->batch_open) {
        e->acc.ms_e2e = now_ms() - e->t0;
        float ms = 0;
        if (e->begun[0] >= 0) {
            e->acc.ms_out = stamped_ms(e, 0);
        } else if (e->b_o0 && e->b_o1) {
            HIPTRY(e, hipEventElapsedTime(&ms, e->b_o0, e->b_o1));
            e->acc.ms_out = ms;
        }
        if (e->begun[1] >= 0) {
            e->acc.ms_in = stamped_ms(e, 1);
        } else if (e->b_i0 && e->b_i1) {
            HIPTRY(e, hipEventElapsedTime(&ms, e->b_i0, e->b_i1));
            e->acc.ms_in = ms;
        }
        e->last = e->acc;
        e->batch_open = false;
    }
    return KV_OK;
}

int kv_query(kv_engine *e)
{
    if (!e) return KV_EINVAL;
    if (e->sticky != KV_OK) return e->sticky;
    for (int side = 0; side < 2; side++) {
        const bool pending = side == 0 ? e->out_pending : e->in_pending;
        if (!pending) continue;
        const hipError_t q = hipStreamQuery(side == 0 ? e->s_out : e->s_in);
        if (q == hipErrorNotReady) {
            (void)hipGetLastError();  // not an error: forget it
            return KV_EBUSY;
        }
        HIPTRY(e, q);
    }
    // nothing runs any more, so nothing can race with what comes next
    e->out_dirty = e->in_dirty = false;
    e->in_behind = nullptr;
    e->hazards.join();
    e->idle_epoch++;
    return KV_OK;
}

// The events behind which `layer` of the most recent transfer call is complete:
// its chunk's events if that call ran layer by layer, else the call's end events.
static int layer_events(kv_engine *e, int32_t layer, hipEvent_t (&out)[2])
{
    out[0] = out[1] = nullptr;
    if (!e || layer < 0 || layer >= e->cfg.n_layers) return KV_EINVAL;
    if (e->sticky != KV_OK) return e->sticky;
    if (e->layer_chunk > 0) {
        const size_t c = (size_t)(layer / e->layer_chunk);
        if (e->layer_on_out) out[0] = e->layer_ev_out[c];
        if (e->layer_on_in) out[1] = e->layer_ev_in[c];
    } else {
        if (e->out_pending) out[0] = e->b_o1;
        if (e->in_pending) out[1] = e->b_i1;
    }
    return KV_OK;
}

int kv_stream_wait_layer(kv_engine *e, void *stream, int32_t layer)
{
    hipEvent_t evs[2];
    const int rc = layer_events(e, layer, evs);
    if (rc != KV_OK) return rc;
    for (hipEvent_t x : evs)
        if (x) HIPTRY(e, hipStreamWaitEvent((hipStream_t)stream, x, 0));
    return KV_OK;
}

int kv_wait_layer(kv_engine *e, int32_t layer)
{
    hipEvent_t evs[2];
    const int rc = layer_events(e, layer, evs);
    if (rc != KV_OK) return rc;
    for (hipEvent_t x : evs)
        if (x) HIPTRY(e, hipEventSynchronize(x));
    return KV_OK;
}

int kv_host_pool(kv_engine *e, void **ptr, uint64_t *bytes)
{
    if (!e || !ptr || !bytes) return KV_EINVAL;
    *ptr = e->pool;
    *bytes = e->pool_bytes;
    return KV_OK;
}

int kv_last_stats(kv_engine *e, kv_stats *out)
{
    if (!e || !out) return KV_EINVAL;
    *out = e->last;
    return KV_OK;
}

int kv_rotate_static(const kv_config *cfg, void *hbm_cache, void *host_pool, void *stream,
                     const int32_t *oi, const int32_t *os, int32_t no, const int32_t *ii, const int32_t *is,
                     int32_t ni)
{
    if (!config_ok(cfg) || !hbm_cache || !host_pool) return KV_EINVAL;
    if (cfg->path != KV_PATH_AUTO && cfg->path != KV_PATH_FUSED) return KV_EUNSUP;
    // the host-side arrays (sorted copies, the argument chunk, the address table) are the
    // process's, not the call's: callers on several threads take turns
    static std::mutex turn;
    std::lock_guard<std::mutex> hold(turn);
    int rc = admit_static(cfg, oi, os, no, ii, is, ni);
    if (rc != KV_OK) return rc;
    // an engine that exists only on this stack frame, so that the launch helpers
    // of the other paths serve here too; nothing in it owns memory
    kv_engine view;
    kv_engine *e = &view;
    e->cfg = *cfg;
    e->seg = seg_of(cfg);
    e->n_planes = 2u * (uint32_t)cfg->n_layers;
    e->block_bytes = kv_block_bytes(cfg);
    e->cache_bytes = kv_cache_bytes(cfg);
    e->pool_bytes = kv_pool_bytes(cfg);
    e->hbm = (uint8_t *)hbm_cache;
    e->pool = (uint8_t *)host_pool;
    e->vec = pick_vec(e);
    // both pointers are checked before a kernel is given them
    {
        hipDeviceptr_t base = nullptr;
        size_t span = 0;
        if (hipMemGetAddressRange(&base, &span, (hipDeviceptr_t)hbm_cache) != hipSuccess ||
            (uintptr_t)hbm_cache + e->cache_bytes > (uintptr_t)base + span) {
            (void)hipGetLastError();
            fprintf(stderr, "duplexkv: hbm_cache is not a device allocation of the configured size\n");
            return KV_EINVAL;
        }
        hipPointerAttribute_t at;
        if (hipPointerGetAttributes(&at, host_pool) != hipSuccess || at.type != hipMemoryTypeHost) {
            (void)hipGetLastError();
            fprintf(stderr, "duplexkv: host_pool is not pinned host memory\n");
            return KV_EINVAL;
        }
        if (hipMemGetAddressRange(&base, &span, (hipDeviceptr_t)host_pool) == hipSuccess) {
            if ((uintptr_t)host_pool + e->pool_bytes > (uintptr_t)base + span) {
                fprintf(stderr, "duplexkv: host_pool allocation is smaller than the configured pool\n");
                return KV_EINVAL;
            }
        } else {
            (void)hipGetLastError();
        }
    }
    if (no == 0 && ni == 0) return KV_OK;
    const LinkKind kind = no == 0 ? kInOnly : ni == 0 ? kOutOnly : ni >= 2 * (int64_t)no ? kInHeavy : kBoth;
    const LinkShape sh = link_shape(e, kind);
    MoveParams p = base_params(e);
    p.fixed_rounds = sh.fixed_rounds;
    p.through = writes_through(e) && sh.through && !leaves_to_l2(e, os, no, ni) ? 1u : 0u;
    p.far_out = p.far_in = e->pool;
    pool_strides(e, p.far_slot_stride_out, p.far_plane_stride_out);
    p.far_slot_stride_in = p.far_slot_stride_out;
    p.far_plane_stride_in = p.far_plane_stride_out;
    p.plane_major = cfg->host_layout == KV_HOST_LAYER_FIRST ? 1u : 0u;
    cut_tiles(p, e->vec, sh.u, piece_align(e, e->n_planes), no > 0);
    if (!fill_dir(p, (uint32_t)no, 0, sh.limit_u, p.out) || !fill_dir(p, (uint32_t)ni, 0, sh.limit_u, p.in))
        return KV_EUNSUP;
    if (p.out.tiles > 0 && p.in.tiles > p.out.tiles)
        p.mix_q = (((uint64_t)p.out.tiles << 32) + p.in.tiles - 1) / p.in.tiles;
    unsigned char *sc = nullptr;
    int dev;
    rc = static_scratch(sc, dev);
    if (rc != KV_OK) return rc;
    p.claim = reinterpret_cast<unsigned int *>(sc);
    int32_t *ids = reinterpret_cast<int32_t *>(sc + kStaticIdsOff);
    hipStream_t s = (hipStream_t)stream;
    static IdChunk chunk;  // one caller at a time
    // Few blocks: the lists are arguments of the one launch.  (1 + 1 blocks of 120 KiB: 31.9 us
    // with the launch that puts them into the array, 28.6 without; 4 + 3 of 2 MiB: 203.6 and 199.6.)
    if (ids_inline(e, no, ni)) {
        if (draws(sh, p)) {
            if (capturing(s)) {
                hipLaunchKernelGGL(kv_ids_kernel, dim3(1), dim3(256), 0, s, chunk, ids, 0u, p.claim);
                HIPTRY((kv_engine *)nullptr, hipGetLastError());
            } else {
                auto pair = [&](int turn) {
                    return reinterpret_cast<unsigned int *>(sc + (size_t)(1 + turn % (kStaticPairs - 1)) * kStaticPairBytes);
                };
                int &turn = g_static_turn[dev];
                p.claim = pair(turn);
                turn = (turn + 1) % (kStaticPairs - 1);
                p.clear = pair(turn);
            }
        }
        launch_move(sh, e->vec, s, p, MoveIds{oi, os, ii, is, true}, true);
        HIPTRY((kv_engine *)nullptr, hipGetLastError());
        return KV_OK;
    }
    // the four lists, back to back, through kernel arguments
    const int32_t *src[4] = {oi, os, ii, is};
    const uint32_t len[4] = {(uint32_t)no, (uint32_t)no, (uint32_t)ni, (uint32_t)ni};
    const uint32_t total = 2u * ((uint32_t)no + (uint32_t)ni);
    uint32_t done = 0, list = 0, at = 0;
    while (done < total) {
        uint32_t n = 0;
        while (n < kIdsPerLaunch && list < 4) {
            const uint32_t take = std::min(kIdsPerLaunch - n, len[list] - at);
            if (take) memcpy(chunk.v + n, src[list] + at, (size_t)take * sizeof(int32_t));
            n += take;
            at += take;
            if (at == len[list]) { list++; at = 0; }
        }
        hipLaunchKernelGGL(kv_ids_kernel, dim3(1), dim3(256), 0, s, chunk, ids + done, n,
                           done == 0 ? p.claim : (unsigned int *)nullptr);
        HIPTRY((kv_engine *)nullptr, hipGetLastError());
        done += n;
    }
    launch_move(sh, e->vec, s, p,
                MoveIds{ids, ids + no, ids + 2 * (size_t)no, ids + 2 * (size_t)no + ni}, true);
    HIPTRY((kv_engine *)nullptr, hipGetLastError());
    return KV_OK;
}

int kv_probe_link(uint64_t bytes, int32_t reps, double *d2h, double *h2d, double *d2h_duplex,
                  double *h2d_duplex)
{
    if (bytes == 0 || reps <= 0 || !d2h || !h2d || !d2h_duplex || !h2d_duplex) return KV_EINVAL;
    kv_engine *e = nullptr;  // HIPTRY wants one; no engine state here
    void *ha = nullptr, *hb = nullptr, *da = nullptr, *db = nullptr;
    // Streams share a few hardware queues and DMA engines; which pair a process
    // gets depends on what else it has created.  Up to three rounds of five
    // streams each (more than the process has hardware queues; earlier rounds'
    // streams stay alive so that later ones land elsewhere): every pairing with
    // a round's first two streams is timed and the best one is reported, the
    // link's ceiling and not a property of one unlucky pairing.  A round that
    // already shows the directions overlapping ends the search.
    constexpr int kS = 5, kRounds = 3;
    hipStream_t st[kS * kRounds] = {};
    auto cleanup = [&]() {
        if (ha) (void)hipHostFree(ha);
        if (hb) (void)hipHostFree(hb);
        if (da) (void)hipFree(da);
        if (db) (void)hipFree(db);
        for (int i = 0; i < kS * kRounds; i++)
            if (st[i]) (void)hipStreamDestroy(st[i]);
    };
    if (hipHostMalloc(&ha, bytes, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc(&hb, bytes, hipHostMallocDefault) != hipSuccess ||
        hipMalloc(&da, bytes) != hipSuccess || hipMalloc(&db, bytes) != hipSuccess) {
        (void)hipGetLastError();
        cleanup();
        return KV_ENOMEM;
    }
    memset(ha, 1, bytes);
    memset(hb, 2, bytes);
    // one timed pass: D2H on `so` and / or H2D on `si`; returns wall ms to the last completion
    auto pass = [&](hipStream_t so, hipStream_t si, double &ms) -> int {
        std::vector<double> t;
        for (int it = 0; it < reps + 2; it++) {
            HIPTRY(e, hipDeviceSynchronize());
            const double a = now_ms();
            if (so) HIPTRY(e, hipMemcpyAsync(ha, da, bytes, hipMemcpyDeviceToHost, so));
            if (si) HIPTRY(e, hipMemcpyAsync(db, hb, bytes, hipMemcpyHostToDevice, si));
            if (so) HIPTRY(e, hipStreamSynchronize(so));
            if (si) HIPTRY(e, hipStreamSynchronize(si));
            if (it >= 2) t.push_back(now_ms() - a);
        }
        ms = median(t);
        return KV_OK;
    };
    auto body = [&]() -> int {
        HIPTRY(e, hipMemset(da, 3, bytes));
        HIPTRY(e, hipMemset(db, 4, bytes));
        double ms = 0, best = 1e30, one_way = 0;
        const int pairs[7][2] = {{0, 1}, {0, 2}, {0, 3}, {0, 4}, {1, 2}, {1, 3}, {1, 4}};
        for (int r = 0; r < kRounds; r++) {
            hipStream_t *q = st + r * kS;
            for (int i = 0; i < kS; i++) HIPTRY(e, hipStreamCreateWithFlags(&q[i], hipStreamNonBlocking));
            if (r == 0) {
                if (pass(q[0], nullptr, ms) != KV_OK) return KV_EHIP;
                *d2h = bytes / ms / 1e6;
                one_way = ms;
                if (pass(nullptr, q[1], ms) != KV_OK) return KV_EHIP;
                *h2d = bytes / ms / 1e6;
                one_way = std::max(one_way, ms);
            }
            for (auto &pr : pairs) {
                if (pass(q[pr[0]], q[pr[1]], ms) != KV_OK) return KV_EHIP;
                best = std::min(best, ms);
            }
            if (best < 1.5 * one_way) break;  // the two copies overlapped
        }
        // both directions are charged the wall time of the pair
        *d2h_duplex = *h2d_duplex = bytes / best / 1e6;
        return KV_OK;
    };
    int rc = body();
    (void)hipDeviceSynchronize();
    cleanup();
    return rc;
}

int kv_reader_start(kv_engine *e, const int32_t *ids, int32_t n, int32_t passes, int32_t max_wgs)
{
    if (!e || list_bad(ids, n) || passes < 1 || passes > kReadPasses || max_wgs < 0) return KV_EINVAL;
    if (e->sticky != KV_OK) return e->sticky;
    if (e->read_passes != 0) return KV_EINVAL;  // previous reader not waited for
    if (out_of_range(ids, n, e->cfg.n_hbm_blocks)) return KV_ERANGE;
    if ((int64_t)n > 2 * (int64_t)e->cfg.n_hbm_blocks) return KV_EINVAL;
    if (e->seg % 16 != 0 || ((uintptr_t)e->hbm & 15u) != 0) return KV_EUNSUP;
    // Workgroups: 5.5 per CU.  With one row in flight per wave (kReadDepth) that is 5.6 MiB
    // in flight, enough for the HBM rate alone, and the most that a copy beside it bears
    // without loss (8 GiB passes, TB/s alone / beside a swap-out, and its GB/s / beside a
    // rotation, and its GB/s): 5 per CU 6.77 / 6.55, 56.9 / 5.19, 101.0;  5.5 7.00 / 6.74, 56.8 /
    // 5.48, 101.0;  6 7.09 / 5.62, 55.4 / 4.50, 98.5;  7 6.41 / 5.77, 55.5 / 4.66, 98.5.
    const int most_wgs = 11 * (e->n_cus > 0 ? e->n_cus : 256) / 2;
    constexpr size_t kReadCounters = (size_t)dkv::kReadGroups * dkv::kReadStride;  // words of one set of counters
    if (!e->s_read) {
        const size_t idb = 2 * (size_t)e->cfg.n_hbm_blocks * sizeof(int32_t);
        if (hipMalloc((void **)&e->read_ids, idb) != hipSuccess ||
            hipHostMalloc((void **)&e->read_ids_host, idb, hipHostMallocDefault) != hipSuccess ||
            hipMalloc((void **)&e->read_part,
                      (size_t)most_wgs * sizeof(unsigned long long) + 2 * kReadCounters * sizeof(unsigned int)) != hipSuccess ||
            hipHostMalloc((void **)&e->read_sums, (2 * (size_t)most_wgs + dkv::kReadBegins) * sizeof(unsigned long long),
                          hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return KV_ENOMEM;
        }
        HIPTRY(e, hipStreamCreateWithFlags(&e->s_read, hipStreamNonBlocking));
        HIPTRY(e, hipMemsetAsync(e->read_part + most_wgs, 0, 2 * kReadCounters * sizeof(unsigned int), e->s_read));
    }
    // One pass is timed by the clock that its workgroups leave (an event ahead of it is a
    // packet that it waits for: 2 MiB 17.3 us with events, 16.2 without, 375 MiB 78.5 and 77.4),
    // several by events between them.
    const bool events = passes > 1;
    while (events && (int32_t)e->read_ev.size() < passes + 1) {
        hipEvent_t x;
        HIPTRY(e, hipEventCreate(&x));
        e->read_ev.push_back(x);
    }
    dkv::ReadParams p{};
    p.hbm = e->hbm;
    p.part = e->read_part;
    p.result = reinterpret_cast<dkv::u64x2 *>(e->read_sums);
    p.passes = (uint32_t)passes;
    hbm_strides(e, p.hbm_plane_stride, p.hbm_block_stride);
    p.n = (uint32_t)n;
    p.vec_per_seg = (uint32_t)(e->seg / 16);
    // the limit on what one pass may name: 2^31 tiles, each within a segment (rows of the
    // flat sequence fit 32 bits then: n is at most twice the blocks there is memory for)
    uint32_t by_segment;
    if (!dir_tiles(p.n, e->n_planes, (p.vec_per_seg + dkv::kReadVecs - 1) / dkv::kReadVecs, by_segment))
        return KV_EUNSUP;
    p.n_vecs = (uint64_t)p.n * e->n_planes * p.vec_per_seg;
    int wgs = most_wgs;
    if (max_wgs > 0) wgs = std::min(wgs, (int)max_wgs);
    constexpr uint32_t waves_per_wg = dkv::kThreads / dkv::kWave;
    const uint64_t n_rows = (p.n_vecs + dkv::kWave - 1) / dkv::kWave;
    const uint64_t each = (n_rows + (uint64_t)wgs * waves_per_wg - 1) / ((uint64_t)wgs * waves_per_wg);  // rows of a wave
    const bool is_short = each <= dkv::kReadShortRows;
    p.rows = (uint32_t)dkv::kReadU;
    if (is_short) {
        const uint32_t rounds = std::max(1u, ((uint32_t)each + dkv::kReadU - 1) / dkv::kReadU);
        p.rows = std::max(1u, ((uint32_t)each + rounds - 1) / rounds);
        p.rows += p.rows % dkv::kReadShortDepth;
    }
    p.tiles = (uint32_t)((n_rows + p.rows * waves_per_wg - 1) / (p.rows * waves_per_wg));
    // a rounded-up reciprocal is exact while index * divisor stays below 2^64 (and 2^64 / 1 has no room)
    if (p.vec_per_seg > 1 && p.n_vecs <= ~0ull / p.vec_per_seg) p.seg_magic = ~0ull / p.vec_per_seg + 1;
    unsigned int *const next = reinterpret_cast<unsigned int *>(e->read_part + most_wgs);
    wgs = (int)std::min<uint32_t>((uint32_t)wgs, std::max<uint32_t>(p.tiles, 1u));
    // Who reads which tile.  Short passes (under four rounds of the grid, 176 MiB): every
    // workgroup takes its fixed share, no counter.  Longer ones: a quarter in fixed shares,
    // the rest claimed from the workgroup's group, and in passes of 64 rounds and more,
    // which a last look at other groups' counters does not lengthen, from two groups behind it.
    // TB/s alone / beside a swap-out / a swap-in / the default rotation, one by 192 waves:
    //   37.5 GiB from no other group 7.04 / 6.80 / 5.34 / 5.47, 4.94, from two 7.04 / 6.82 / 5.38 / 5.52, 4.94
    //    8   GiB                     7.02 / 6.74 / 5.38 / 5.38, 4.92           7.01 / 6.75 / 5.41 / 5.48, 4.91
    //    2   GiB                     6.70 / 6.46 / 5.48 / 5.53, 4.46           6.68 / 6.44 / 5.51 / 5.66, 4.43
    //    256 MiB                     5.43 / 4.99 / 4.23 / 4.19, 3.37           5.39 / 4.80 / 4.08 / 3.98, 2.83
    // Beside swap-outs that slowed it more (their stores went through the L2), an eighth or a
    // sixteenth in fixed shares changed nothing beyond 2 %; with half or all fixed,
    // workgroups that a copy slows set the pace (all: 2.9 TB/s beside a swap-out of 4 GiB).
    // Under four rounds that is over before it matters: 90 and 160 MiB take 23 and 33 us alone,
    // 30 and 41 beside a swap-out, 42 and 59 beside a rotation.
    const uint32_t rounds = p.tiles / (uint32_t)wgs;
    p.fixed = rounds < 4 ? rounds + 1 : rounds / 4;
    p.steal = rounds < 64 ? 0 : 2;
    const bool rows = p.vec_per_seg % dkv::kWave == 0;
    dkv::IdArgs a;
    const bool singly = n <= (int32_t)dkv::kInlineIds;
    const bool pairs = !singly && n <= 2 * (int32_t)dkv::kInlineIds && e->cfg.n_hbm_blocks <= 65536;
    if (singly) {
        std::copy(ids, ids + n, a.v);
    } else if (pairs) {
        for (int32_t i = 0; i + 1 < n; i += 2) a.v[i / 2] = (int32_t)((uint32_t)ids[i] | (uint32_t)ids[i + 1] << 16);
        if (n % 2) a.v[n / 2] = ids[n - 1];
    } else {
        memcpy(e->read_ids_host, ids, (size_t)n * sizeof(int32_t));
        const unsigned g = std::min(64u, ((unsigned)n + dkv::kThreads - 1) / dkv::kThreads);
        hipLaunchKernelGGL(dkv::kv_reader_ids_kernel, dim3(g), dim3(dkv::kThreads), 0, e->s_read, e->read_ids_host,
                           e->read_ids, p.n);
        HIPTRY(e, hipGetLastError());
    }
    if (events) HIPTRY(e, hipEventRecord(e->read_ev[0], e->s_read));
    else p.begin = e->read_sums + 2 * (size_t)wgs;
    for (int32_t k = 0; k < passes; k++) {
        if (p.tiles > 0) {
            p.pass = (uint32_t)k;
            p.next = next + e->read_turn * kReadCounters;
            p.clear = next + (1 - e->read_turn) * kReadCounters;
            e->read_turn = 1 - e->read_turn;
            const dim3 g((unsigned)wgs), b(dkv::kThreads);
            auto go = [&](auto has_rows, auto is_short_pass) {
                constexpr bool R = decltype(has_rows)::value, S = decltype(is_short_pass)::value;
                if (singly) launch(dkv::kv_reader_inline_kernel<R, S, dkv::IdsInArgs>, g, b, e->s_read, nullptr, p, a);
                else if (pairs) launch(dkv::kv_reader_inline_kernel<R, S, dkv::IdPairsInArgs>, g, b, e->s_read, nullptr, p, a);
                else launch(dkv::kv_reader_kernel<R, S>, g, b, e->s_read, nullptr, p, (const int32_t *)e->read_ids);
            };
            const std::true_type yes;
            const std::false_type no;
            if (rows && is_short) go(yes, yes);
            else if (rows) go(yes, no);
            else if (is_short) go(no, yes);
            else go(no, no);
            HIPTRY(e, hipGetLastError());
        }
        if (events) HIPTRY(e, hipEventRecord(e->read_ev[(size_t)k + 1], e->s_read));
    }
    e->read_wgs = p.tiles > 0 ? wgs : 0;
    e->read_passes = passes;
    return KV_OK;
}

int kv_reader_wait(kv_engine *e, uint64_t *checksum, double *ms_per_pass)
{
    if (!e || !checksum) return KV_EINVAL;
    if (e->sticky != KV_OK) return e->sticky;
    if (e->read_passes == 0) return KV_EINVAL;
    HIPTRY(e, hipStreamSynchronize(e->s_read));
    uint64_t sum = 0, begin = ~0ull, end = 0;
    for (int w = 0; w < e->read_wgs; w++) {
        sum += e->read_sums[2 * w];
        end = std::max<uint64_t>(end, e->read_sums[2 * w + 1]);
        if (e->read_passes == 1 && w < (int)dkv::kReadBegins) begin = std::min<uint64_t>(begin, e->read_sums[2 * e->read_wgs + w]);
    }
    *checksum = sum;
    if (ms_per_pass && e->read_passes == 1) {
        ms_per_pass[0] = e->read_wgs ? (double)(end - begin) * e->stamp_ms : 0.0;
    } else if (ms_per_pass) {
        for (int32_t k = 0; k < e->read_passes; k++) {
            float ms = 0;
            HIPTRY(e, hipEventElapsedTime(&ms, e->read_ev[(size_t)k], e->read_ev[(size_t)k + 1]));
            ms_per_pass[k] = ms;
        }
    }
    e->read_passes = 0;
    return KV_OK;
}

const char *kv_strerror(int code)
{
    switch (code) {
    case KV_OK: return "ok";
    case KV_EINVAL: return "invalid argument or configuration";
    case KV_ERANGE: return "block id or host slot out of range";
    case KV_EDUP: return "duplicate id within one list";
    case KV_EOVERLAP: return "block or slot named for both directions";
    case KV_ENOMEM: return "allocation failed";
    case KV_EHIP: return "HIP runtime failure";
    case KV_EUNSUP: return "path cannot serve this shape or request";
    case KV_EBUSY: return "block or slot still in use by an un-waited call on the other stream";
    case KV_ENOSPC: return "not enough free HBM blocks or host slots";
    case KV_E2BIG: return "more blocks than the allocation-free entry point's scratch array holds";
    default: return "unknown code";
    }
}

}  // extern "C"
