// Device kernels of the KV rotation engine (gfx950, wave64).
//
// Everything here is data movement: no MFMA, no arithmetic beyond addressing.
// One kernel family, kv_move_kernel, serves every use:
//   - duplex rotation in ONE launch: each lane alternates a 16-byte move
//     HBM->host with a 16-byte move host->HBM, which keeps the two PCIe
//     directions locked 1:1 (measured faster in duplex than two independent
//     kernels, and above the DMA engines' duplex rate);
//   - a single direction (the other list empty): zero-copy swap-out or swap-in;
//     (both also as kv_move_inline_kernel, few blocks, lists in the arguments)
//   - pack / unpack between the scattered cache and a contiguous staging
//     buffer in HBM (the "far" side is then device memory, slot = list index)
//     when the launch is capped to a few workgroups; uncapped, pack / unpack
//     have a kernel of their own, kv_stage_kernel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dkv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));

// Id lists of a call that names few blocks, handed over as a kernel argument: the
// runtime keeps arguments where the device reads them like its own memory.  From
// pinned host memory the first ids of a launch cost it a round trip over the
// link before its first byte moves (2-6 us), and a launch or copy that brings
// them to device memory costs 5.
constexpr uint32_t kInlineIds = 896;  // 3.5 of the 4 KiB that a kernel's arguments may take
struct IdArgs {
    int32_t v[kInlineIds];
};

// Entry i of a reader's list: in device memory, in the arguments, or there two ids to a
// word, which makes room for twice as many where the cache has no more than 65536 blocks.
// (Only where that is needed: taking the words apart costs a pass over 64 MiB 0.9 of 18 us.)
// word() is what is loaded for it, id() takes it out of that: all words of a tile are
// asked for before the first is taken apart.  Taken apart where they are loaded, each was
// waited for by itself: 995 blocks of 100 x 2688 bytes, where every lane fetches its own, in
// 63.6 us and now 46.7 (a call 78.4 and 61.4).
struct IdsInMemory {
    const int32_t *__restrict__ ids;
    __device__ __forceinline__ uint32_t word(uint32_t i) const { return (uint32_t)ids[i]; }
    static __device__ __forceinline__ uint32_t id(uint32_t w, uint32_t) { return w; }
};
struct IdsInArgs {
    const IdArgs &a;
    __device__ __forceinline__ uint32_t word(uint32_t i) const { return (uint32_t)a.v[i]; }
    static __device__ __forceinline__ uint32_t id(uint32_t w, uint32_t) { return w; }
};
struct IdPairsInArgs {
    const IdArgs &a;
    __device__ __forceinline__ uint32_t word(uint32_t i) const { return (uint32_t)a.v[i >> 1]; }
    static __device__ __forceinline__ uint32_t id(uint32_t w, uint32_t i) { return w >> ((i & 1u) * 16u) & 0xFFFFu; }
};

constexpr int kWave = 64;          // a wave is the unit of work: one tile at a time
constexpr int kThreads = 256;      // lanes per workgroup of the HBM-bound launches and of the reader (4 waves)
// Vectors per lane where a tile may span segments: every vector has pointers of its
// own there, and with eight they would not fit the registers of a 1024-lane workgroup.
constexpr int kMaxRaggedU = 4;
constexpr uint32_t kStretch = 256;  // bytes of the far side that tiles begin on a multiple of (MoveParams::line_mask)
// Places for the time stamps of a launch, one per wave: at least as many as any launch shape
// that the engine picks has waves.  (Of more, w and w + kStamps share one; the wave that
// ends later stores later.)
constexpr uint32_t kStamps = 512;
constexpr int kMaxThreads = 1024;  // workgroups only pack waves; any multiple of 64 up to this

// Division by a number that is the same for a whole launch, x < 2^31: a multiply
// and a shift by host-made constants, on the scalar unit where x is uniform.  (The
// compiler's own division is ~25 vector instructions; a step has up to six.)
struct Div {
    uint32_t d, m, s;
    __device__ __forceinline__ uint32_t quotient(uint32_t x) const { return __umulhi(x << 1, m) >> s; }
};

inline Div make_div(uint32_t d)  // 1 <= d < 2^31
{
    uint32_t s = 0;
    while ((1u << s) < d) s++;
    return Div{d, (uint32_t)(((1ull << (31 + s)) + d - 1) / d), s};  // x * (m * d - 2^(31+s)) < 2^31 * d <= 2^(31+s)
}

// One direction's block list as the kernel sees it.  The id arrays themselves
// are separate __restrict__ kernel arguments so that the compiler fetches them
// with scalar loads (their own counter, off the vector-memory critical path).
struct DirDesc {
    uint32_t n;      // blocks
    uint32_t tiles;  // n * groups_per_entry * tiles_per_group
    uint32_t iota;   // 1: far-side slot of list entry i is i itself (staging); 0: slots[i]
    Div inner;       // by the faster of the two group indices' range: plane-major n, else groups_per_entry
};

// Addressing (Section 4.3.1 of the paper: layer x block x segment):
//   HBM  segment (plane, id)   at hbm + plane * hbm_plane_stride + id * hbm_block_stride
//   far  segment (plane, slot) at far + slot * far_slot_stride + plane * far_plane_stride
// `plane` = layer * 2 + (0 for K, 1 for V).
struct MoveParams {
    uint8_t *hbm;
    uint8_t *far_out;  // destination of the out direction (host pool or staging)
    uint8_t *far_in;   // source of the in direction
    uint64_t hbm_plane_stride;  // layer-first cache: blocks * seg; block-first cache: seg
    uint64_t hbm_block_stride;  // layer-first cache: seg;          block-first cache: planes * seg
    uint64_t far_slot_stride_out, far_plane_stride_out;
    uint64_t far_slot_stride_in, far_plane_stride_in;
    uint32_t plane0;         // first plane this launch covers
    uint32_t n_planes;       // planes this launch covers
    uint32_t vec_per_seg;    // segment bytes / sizeof(V)
    // A group is what tiles are cut from: one segment, or (segments that are no whole
    // number of tiles, far side [i][plane]...) all segments of a list entry, which
    // are one range on the far side and planes apart in the cache.
    uint32_t group_vecs;        // vec_per_seg, or n_planes * vec_per_seg
    uint32_t groups_per_entry;  // n_planes, or 1
    // Tiles begin on stretches of kStretch bytes of the far side, so that only the first and the
    // last access of a group cover part of one: 0 where groups begin on stretches anyway, else
    // the vectors of a stretch - 1; the first tile then holds as many vectors fewer as the
    // group begins behind one.  A write on the link carries up to 256 bytes, none across a multiple of 256: an
    // access of 1 KiB that begins on an odd line is five of them instead of four.  (Layer-first
    // pool, 24 MiB both ways / out / in, us, tiles on 128-byte lines and on stretches: 2400-byte segments
    // 533 / 464 / 461 and 513 / 447 / 458, 2688 bytes 523 / 460 / 446 and 503 / 442 / 439, 1600 bytes 526 / 462 /
    // 459 and 515 / 448 / 459; blocks of 28800 bytes, block-first, 521 / 458 / 450 and 505 / 443 / 440.  Taken as
    // they lie, 3360-byte segments, 40 MiB, lost another 15 / 5 / 0.)
    uint32_t line_mask;
    Div by_tiles;               // by tiles_per_group = ceil((group_vecs + line_mask) / (64 * U))
    Div by_seg;                 // by vec_per_seg (quotient 0 where a group is one segment)
    uint32_t plane_major;       // group order: 1 = [plane][i], 0 = [i][plane]
    uint32_t through;           // vectors of 8 bytes and more: 1 = written through to the host (store_host)
    uint32_t full_tiles;        // 1: a group is one segment, taken in whole tiles
    uint64_t plane_skip;        // cache bytes between the end of a segment and the same block's next one
    // 0, or ceil(out.tiles * 2^32 / in.tiles) when the in list is the longer one and
    // the out tiles are to be spread evenly over it (see make_job)
    uint64_t mix_q;
    // link-bound launches: two counters in device memory, zero at launch, [0] the
    // next unclaimed tile, [1] the waves that are done
    unsigned int *claim;
    unsigned int *clear;  // nullptr, or a pair that a later launch draws from: put to zero
    // Pinned host memory, or nullptr: where each wave w leaves the device's clock, in
    // stamps[w % kStamps], as it was when the wave began, and when it ended, with `drain` when
    // its last store has arrived.  The launch begins with its first wave, whichever that is:
    // beside a launch on another stream, wave 0 was up to 19 us later.
    u64x2 *stamps;
    uint32_t drain;
    uint32_t fixed_rounds;  // link-bound launches of at most this many steps per wave take fixed shares
    DirDesc out, in;
};


// Tile t of direction d -> byte offsets of its group on both sides, and its place
// within the group.
__device__ __forceinline__ void locate(const MoveParams &p, const DirDesc &d,
                                       const int32_t *__restrict__ ids,
                                       const int32_t *__restrict__ slots, uint32_t t,
                                       uint64_t slot_stride, uint64_t plane_stride,
                                       uint64_t &hbm_off, uint64_t &far_off, uint32_t &tin)
{
    const uint32_t group = p.by_tiles.quotient(t);
    tin = t - group * p.by_tiles.d;
    const uint32_t q = d.inner.quotient(group), r = group - q * d.inner.d;
    const uint32_t i = p.plane_major ? r : q, pl = p.plane0 + (p.plane_major ? q : r);
    const uint32_t id = (uint32_t)ids[i];
    const uint32_t slot = d.iota ? i : (uint32_t)slots[i];
    hbm_off = (uint64_t)pl * p.hbm_plane_stride + (uint64_t)id * p.hbm_block_stride;
    far_off = (uint64_t)slot * slot_stride + (uint64_t)pl * plane_stride;
}

// What one wave does in one step: an in tile, an out tile, or one of each.
// The lane's pointers are worked out a step ahead, all of them: an address
// computed where its load is issued lands in a register of the step before, and
// the wave waits for that step's accesses first.  In a FULL tile one pointer per
// side serves all vectors of the lane; elsewhere the group may continue in
// another plane of the cache, or end.
template <typename V, int U, bool FULL>
struct Job {
    static constexpr int N = FULL ? 1 : U;
    const V *src_i[N];
    V *dst_i[N];
    const V *src_o[N];
    V *dst_o[N];
    uint32_t do_in, do_out;
    uint32_t n_i, n_o;  // vectors of the group from this lane's first one on (not FULL: what the stores go by)
};

// The lane's pointers into one tile; past the end of the group, to its last vector,
// before its begin, to its first (with the same value: these lanes are not told apart).
template <typename V, int U, bool FULL, int N>
__device__ __forceinline__ void lane_pointers(const MoveParams &p, uint64_t hbm_off, uint8_t *far, uint32_t tin,
                                              uint32_t lane, V *(&in_cache)[N], V *(&in_far)[N], uint32_t &n)
{
    uint32_t v0 = tin * (kWave * U) + lane;
    bool before = false;
    if constexpr (!FULL) {
        const uint32_t begin = (uint32_t)(reinterpret_cast<uintptr_t>(far) / sizeof(V)) & p.line_mask;
        before = v0 < begin;
        v0 -= begin;
    }
    n = p.group_vecs - v0;
#pragma unroll
    for (int u = 0; u < N; u++) {
        uint32_t v = v0 + u * kWave;
        uint64_t off = hbm_off;
        if constexpr (!FULL) {
            v = min(u == 0 && before ? 0u : v, p.group_vecs - 1u);
            off += (uint64_t)p.by_seg.quotient(v) * p.plane_skip;
        }
        in_cache[u] = reinterpret_cast<V *>(p.hbm + off) + v;
        in_far[u] = reinterpret_cast<V *>(far) + v;
    }
    if (!before && v0 >= p.group_vecs) n = 0u;
}

// Step t of a launch.  Normally step t is tile t of the out list and tile t of
// the in list, as far as each list goes: while both last, every lane alternates
// an out-vector with an in-vector, which locks the two link directions 1:1, and
// the longer list's remainder then runs alone.
//
// With mix_q set the in list is the longer one: its tiles set the pace and the
// out tiles are spread evenly over them, out tile s riding with the in tile t
// at which floor(t * q / 2^32) steps from s to s + 1 (q = ceil(S * 2^32 / L), so
// the steps are 0 or 1 and all S out tiles are met exactly once over the L in
// tiles).  Measured on PCIe Gen5 x16: host->HBM reads can stay at the link's
// one-way rate (55-57 GB/s) while up to ~0.85 as many bytes go the other way
// (47 GB/s), 102 GB/s in all, whereas pairing the lists 1:1 and moving the rest
// of the in list afterwards holds both at 49.5 GB/s for the paired part.  (The
// mirror case gains nothing: with the out list longer, what limits is the
// upstream direction, which carries the out data and the read requests of the
// in data, and that sum does not depend on the order.)
template <typename V, int U, bool FULL>
__device__ __forceinline__ Job<V, U, FULL> make_job(const MoveParams &p, const int32_t *__restrict__ out_ids,
                                                    const int32_t *__restrict__ out_slots,
                                                    const int32_t *__restrict__ in_ids,
                                                    const int32_t *__restrict__ in_slots, uint32_t t, uint32_t lane)
{
    Job<V, U, FULL> j{};
    constexpr int N = Job<V, U, FULL>::N;
    uint32_t t_out = t;
    if (p.mix_q) {
        const uint64_t a = (uint64_t)t * p.mix_q, b = a + p.mix_q;
        const uint32_t s0 = (uint32_t)(a >> 32);
        uint32_t s1 = (uint32_t)(b >> 32);
        s1 = s1 < p.out.tiles ? s1 : p.out.tiles;
        j.do_in = 1u;
        j.do_out = s1 > s0 ? 1u : 0u;
        t_out = s0;
    } else {
        j.do_in = t < p.in.tiles ? 1u : 0u;
        j.do_out = t < p.out.tiles ? 1u : 0u;
    }
    uint64_t ho, fo;
    uint32_t tin;
    if (j.do_in) {
        locate(p, p.in, in_ids, in_slots, t, p.far_slot_stride_in, p.far_plane_stride_in, ho, fo, tin);
        V *far[N];
        lane_pointers<V, U, FULL, N>(p, ho, p.far_in + fo, tin, lane, j.dst_i, far, j.n_i);
#pragma unroll
        for (int u = 0; u < N; u++) j.src_i[u] = far[u];
    }
    if (j.do_out) {
        locate(p, p.out, out_ids, out_slots, t_out, p.far_slot_stride_out, p.far_plane_stride_out, ho, fo, tin);
        V *cache[N];
        lane_pointers<V, U, FULL, N>(p, ho, p.far_out + fo, tin, lane, cache, j.dst_o, j.n_o);
#pragma unroll
        for (int u = 0; u < N; u++) j.src_o[u] = cache[u];
    }
    return j;
}

// Loads of one job: the far-side (host) loads first, they have the long
// latency; then the HBM loads.  Lanes past the group's end load nothing from the
// host (a vector that many lanes repeat crosses the link once for every 16 of
// them), and repeat the group's last vector from HBM.  In an HBM-bound launch (pack / unpack, !LINK)
// loads and stores alike are marked non-temporal: nothing a mover touches is
// touched twice.
template <typename V, int U, bool LINK, bool FULL>
__device__ __forceinline__ void job_loads(const Job<V, U, FULL> &j, V (&vi)[U], V (&vo)[U])
{
    if (j.do_in) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const V *src = FULL ? j.src_i[0] + u * kWave : j.src_i[FULL ? 0 : u];
            if constexpr (!LINK) vi[u] = __builtin_nontemporal_load(src);
            else if (FULL || (uint32_t)(u * kWave) < j.n_i) vi[u] = *src;
        }
    }
    if (j.do_out) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const V *src = FULL ? j.src_o[0] + u * kWave : j.src_o[FULL ? 0 : u];
            if constexpr (LINK) vo[u] = *src;
            else vo[u] = __builtin_nontemporal_load(src);
        }
    }
}

// A vector to host memory.  16-byte vectors are written through ("system" scope), so
// they leave the chip when they are stored.  Stores that end in the write-back L2,
// non-temporal ones too, are taken in at 90 GB/s until ~3 MiB of them lie there:
// the link upstream idles meanwhile, and the kernel's end waits until the rest is
// pushed out at less than the link's rate.  Written through, a store is acknowledged
// from the host's side, so the waves are paced by the link and need no tuning for it
// (from 64 KiB in flight on every shape moves 57.1 GB/s out, where 112 waves of
// non-temporal stores came to 55.8), the L2 stays the other kernels', and an HBM-bound
// reader beside a swap-out keeps 6.8 instead of 6.5 TB/s.  Kernel time in us, plain /
// non-temporal / written through: out 0.5 MiB 18.7 / 18.6 / 13.6, 2 MiB 64 / 58 / 41,
// 256 MiB 4890 / 4813 / 4700; both ways 2 MiB each 79 / 73 / 48, 256 MiB 5418 / 5341 / 5320.
// So do 8-byte vectors (40 MiB both ways, us, non-temporal / written through: 840-byte segments
// in a block-first pool 901 / 853).  Every part of a line is a write of its own on the link,
// though, where the L2 would have joined them: vectors of 4 bytes and less (180-byte segments
// 1187 / 1557) are never written through, and wider ones not in the calls that
// leaves_to_l2() names.
template <typename V, bool THROUGH>
__device__ __forceinline__ void store_host(const V &v, V *dst)
{
    if constexpr (THROUGH && sizeof(V) == 16) {
        __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) u32x4 *)dst, v, "");
    } else if constexpr (THROUGH) {
        static_assert(sizeof(V) == 8);
        __scoped_atomic_store_n(reinterpret_cast<uint64_t *>(dst), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                                __MEMORY_SCOPE_SYSTEM);
    } else {
        __builtin_nontemporal_store(v, dst);
    }
}

// Stores of one job.  Stores to host memory: store_host.  Into the cache, LINK: plain
// stores.  Pack / unpack (both sides HBM): non-temporal, one 256 MiB chunk whose source
// is in no cache with plain loads and stores 109 us, with non-temporal stores 100 us,
// with non-temporal loads and stores 95 us (HIP events around the launch).
template <typename V, int U, bool THROUGH, bool FULL>
__device__ __forceinline__ void out_stores(const Job<V, U, FULL> &j, const V (&vo)[U])
{
#pragma unroll
    for (int u = 0; u < U; u++) {
        V *dst = FULL ? j.dst_o[0] + u * kWave : j.dst_o[FULL ? 0 : u];
        if (FULL || (uint32_t)(u * kWave) < j.n_o) store_host<V, THROUGH>(vo[u], dst);
    }
}

template <typename V, int U, bool LINK, bool FULL>
__device__ __forceinline__ void job_stores(const Job<V, U, FULL> &j, const V (&vi)[U], const V (&vo)[U], uint32_t through)
{
    if (j.do_out) {
        constexpr bool can = LINK && sizeof(V) >= 8;
        if (can && through) out_stores<V, U, can, FULL>(j, vo);
        else out_stores<V, U, false, FULL>(j, vo);
    }
    if (j.do_in) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            V *dst = FULL ? j.dst_i[0] + u * kWave : j.dst_i[FULL ? 0 : u];
            if (FULL || (uint32_t)(u * kWave) < j.n_i) {
                if constexpr (LINK) *dst = vi[u];
                else __builtin_nontemporal_store(vi[u], dst);
            }
        }
    }
}

// One draw of `n` consecutive steps from the counter by the wave's first lane
// (the others get 0).  The value comes back a memory latency later; drawn()
// reads it.
__device__ __forceinline__ uint32_t draw(const MoveParams &p, uint32_t lane, uint32_t n)
{
    uint32_t d = 0;
    if (lane == 0) d = atomicAdd(&p.claim[0], n);
    return d;
}

// The drawn value, wave-uniform.  The empty asm pins the first use of the
// register to this point of the program: without it the compiler is free to
// read the value (and so to wait for the atomic and for every vector memory
// access issued before it) right behind the draw.
__device__ __forceinline__ uint32_t drawn(uint32_t d)
{
    asm volatile("" : "+v"(d));
    return __builtin_amdgcn_readfirstlane(d);
}

// Fixed share: wave w of W takes steps w, w + W, ...  HBM-bound launches, and link-bound
// ones of at most MoveParams::fixed_rounds steps per wave, which the host sets: kFixedRounds where a
// launch carries one direction (1.5 MiB out, 2.25 in, by the default shapes of whole tiles),
// kFixedRoundsBoth where it carries two (1.1 MiB); two launches beside one another: see run_zero_copy().
// In those the waves have no time to drift apart, and the counter's atomics, ~14 ns
// each on one address and slower beside a kernel that fills the memory's queues, are no small part of
// the launch.  With shares to 8, 16 and 24 rounds one way, us a call alone, and beside a reader over 8 GiB with
// the ms that it loses per GiB moved: 1.5 MiB out 42.9, 42.6, 42.3 and 48.4 (1.34), 48.2 (1.32), 45.0 (1.10);
// 1.4 MiB in 42.2, 41.6, 41.6 and 49.2 (2.28), 44.4 (2.31), 44.4; 2 MiB in 53.1, 53.0, 53.2 and 60.6 (2.10), 60.5
// (2.08), 56.0 (2.13).  Both ways, where a step is two tiles, the waves drift further apart, and what more shares
// are worth alone goes by the call: with shares to 8, 12 and 16 rounds one block of 1.3 MiB 44.7, 45.1, 45.0, 80 of
// 16 KiB 44.7, 44.5, 44.3, one of 2 MiB 59.2, 59.2, 59.6.  (Beside the reader they would be 5 to 8 % faster, the one
// block 50.8 (1.40), 47.3 (1.52), 47.3 (1.54).  A wave per step, up to 512 of them, cost the reader half.)
constexpr uint32_t kFixedRounds = 24, kFixedRoundsBoth = 8;

template <typename V, int U, bool LINK, bool FULL>
__device__ __forceinline__ void run_fixed(const MoveParams &p, const int32_t *__restrict__ out_ids,
                                          const int32_t *__restrict__ out_slots,
                                          const int32_t *__restrict__ in_ids,
                                          const int32_t *__restrict__ in_slots, uint32_t n_steps, uint32_t wave,
                                          uint32_t n_waves, uint32_t lane)
{
    uint32_t t = wave;
    if (t >= n_steps) return;
    V vi[U], vo[U];
    Job<V, U, FULL> cur = make_job<V, U, FULL>(p, out_ids, out_slots, in_ids, in_slots, t, lane);
    for (;;) {
        job_loads<V, U, LINK, FULL>(cur, vi, vo);
        t += n_waves;
        const bool more = t < n_steps;
        Job<V, U, FULL> nxt = cur;
        if (more) nxt = make_job<V, U, FULL>(p, out_ids, out_slots, in_ids, in_slots, t, lane);
        job_stores<V, U, LINK, FULL>(cur, vi, vo, p.through);
        if (!more) break;
        cur = nxt;
    }
}

// Drawn steps.  Wave w begins with step w; the steps from n_waves on are drawn from
// p.claim[0], which counts them from there.  A draw takes kDrawChunk consecutive
// steps (one atomic per step would be ~50 M a second on one address, which beside
// an HBM-bound kernel is what limits the launch: 93 GB/s whatever the number of
// waves), except near the end, where steps are drawn singly so that the waves
// still finish within one step of each other.  The draw for the next chunk is issued when the current
// chunk starts and read when it ends.
//
// Every draw the wave issued has been read back when it finds no step left, so
// the counter holds all of its increments before the wave reports itself done in
// p.claim[1]; the wave that sees every other one done puts both back to zero for
// the next launch on the stream.
constexpr uint32_t kDrawChunk = 4;

template <typename V, int U, bool LINK, bool FULL>
__device__ __forceinline__ void run_drawn(const MoveParams &p, const int32_t *__restrict__ out_ids,
                                          const int32_t *__restrict__ out_slots,
                                          const int32_t *__restrict__ in_ids,
                                          const int32_t *__restrict__ in_slots, uint32_t n_steps, uint32_t wave,
                                          uint32_t n_waves, uint32_t lane)
{
    V vi[U], vo[U];
    Job<V, U, FULL> cur = make_job<V, U, FULL>(p, out_ids, out_slots, in_ids, in_slots, wave, lane);
    // steps at or beyond `single` are drawn one at a time
    const uint32_t tail = 2u * kDrawChunk * n_waves, single = n_steps > tail ? n_steps - tail : 0u;
    uint32_t t = wave, e = wave + 1u;  // current step, end of the chunk it belongs to
    uint32_t cn = n_waves < single ? kDrawChunk : 1u;
    uint32_t d = draw(p, lane, cn);    // the next chunk, in flight
    for (;;) {
        job_loads<V, U, LINK, FULL>(cur, vi, vo);
        // The next step.  At the end of a chunk the pending draw is read: here,
        // where the loads have to be waited for anyway (the draw is older than
        // they are), and before the stores: the vector memory counter retires in
        // order, so reading it behind the stores would wait for them, and a wave
        // would then pay store latency and load latency in turn.  As it is, a
        // step's stores have the whole next step to retire.
        uint32_t tn = t + 1u;
        if (tn >= e) {
            tn = n_waves + drawn(d);
            e = tn + cn;
            cn = tn < single ? kDrawChunk : 1u;
            if (tn < n_steps) d = draw(p, lane, cn);
        }
        const bool more = tn < n_steps;
        Job<V, U, FULL> nxt = cur;
        if (more) nxt = make_job<V, U, FULL>(p, out_ids, out_slots, in_ids, in_slots, tn, lane);
        job_stores<V, U, LINK, FULL>(cur, vi, vo, p.through);
        if (!more) break;
        cur = nxt;
        t = tn;
    }
    (void)drawn(d);  // still in flight if the last chunk ran past the last step
    if (lane == 0 && atomicAdd(&p.claim[1], 1u) == n_waves - 1u) {
        p.claim[0] = 0u;
        p.claim[1] = 0u;
    }
}

// V: vector moved per lane (16 bytes when the segment allows it).
// U: vectors per lane per tile; a tile is 64 * U consecutive vectors of a group
//    (MoveParams), so every wave access touches 64 * sizeof(V) contiguous bytes on
//    the far side, and on the cache's but where a segment ends.
// LINK: the far side is host memory.
// A wave is the unit of work: it takes a step, issues its loads, works out the
// addresses of its next step (two divisions, the scalar loads of id and slot)
// while they are in flight, and stores.  What keeps the link busy is the number
// of waves: a second step in flight per wave buys what a second wave buys.
//
// Which step a wave takes next: in link-bound launches of more than a few rounds the
// waves draw step indices from a counter (the draw for the step after next is issued
// a whole step ahead, so its latency is never waited for).  With a fixed share per
// wave the waves of such a launch drift apart by several per cent and the launch ends
// with a tail of ~100 us in which too few waves are left to fill the link; drawn steps
// end within one tile of each other, and the rate no longer depends on how the
// wave count divides the tile count.  The last wave to finish puts both
// counters back to zero for the next launch on the stream.  HBM-bound launches
// (pack / unpack with a cap on their workgroups; uncapped they run as
// kv_stage_kernel) move a tile in ~2 ns chip-wide, too fast for one counter, and
// use the fixed share, and so do short link-bound ones (run_fixed).
template <typename V, int U, bool LINK>
__device__ __forceinline__ void move(const MoveParams &p, const int32_t *__restrict__ out_ids,
                                     const int32_t *__restrict__ out_slots, const int32_t *__restrict__ in_ids,
                                     const int32_t *__restrict__ in_slots)
{
    const unsigned long long began = LINK ? wall_clock64() : 0;  // stored at the end: here the loads would wait for it
    const uint32_t lane = threadIdx.x & (kWave - 1u), waves_per_wg = blockDim.x / kWave;
    const uint32_t wave = blockIdx.x * waves_per_wg + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t n_waves = gridDim.x * waves_per_wg;
    if (LINK && p.clear && blockIdx.x == 0 && threadIdx.x < 2) p.clear[threadIdx.x] = 0u;
    const uint32_t n_steps = p.mix_q ? p.in.tiles : (p.out.tiles > p.in.tiles ? p.out.tiles : p.in.tiles);
    constexpr int UR = U < kMaxRaggedU ? U : kMaxRaggedU;  // what cut_tiles() cut by when tiles are not whole
    if (!LINK || n_steps <= (uint64_t)p.fixed_rounds * n_waves) {
        if (p.full_tiles)
            run_fixed<V, U, LINK, true>(p, out_ids, out_slots, in_ids, in_slots, n_steps, wave, n_waves, lane);
        else
            run_fixed<V, UR, LINK, false>(p, out_ids, out_slots, in_ids, in_slots, n_steps, wave, n_waves, lane);
    } else if (p.full_tiles) {
        run_drawn<V, U, LINK, true>(p, out_ids, out_slots, in_ids, in_slots, n_steps, wave, n_waves, lane);
    } else {
        run_drawn<V, UR, LINK, false>(p, out_ids, out_slots, in_ids, in_slots, n_steps, wave, n_waves, lane);
    }
    // Time stamps that a launch leaves by itself cost it nothing before it begins; an event
    // recorded ahead of it is a packet of its own, 2 us that the launch waits for.
    if (LINK && p.stamps) {
        if (p.drain) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const unsigned long long now = wall_clock64();
        if (lane == 0) store_host<u32x4, true>(__builtin_bit_cast(u32x4, u64x2{began, now}), reinterpret_cast<u32x4 *>(p.stamps + wave % kStamps));
    }
}

template <typename V, int U, bool LINK>
__global__ __launch_bounds__(kMaxThreads) void kv_move_kernel(const MoveParams p,
                                                              const int32_t *__restrict__ out_ids,
                                                              const int32_t *__restrict__ out_slots,
                                                              const int32_t *__restrict__ in_ids,
                                                              const int32_t *__restrict__ in_slots)
{
    move<V, U, LINK>(p, out_ids, out_slots, in_ids, in_slots);
}

static_assert(sizeof(MoveParams) + sizeof(IdArgs) <= 4096);  // what a kernel's arguments may take

// The lists, back to back, in the arguments: out ids, out slots, in ids, in slots.
template <typename V, int U>
__global__ __launch_bounds__(kMaxThreads) void kv_move_inline_kernel(const MoveParams p, const IdArgs a)
{
    move<V, U, true>(p, a.v, a.v + p.out.n, a.v + 2 * p.out.n, a.v + 2 * p.out.n + p.in.n);
}

// Pack / unpack of the DMA-staged path when nothing caps the launch: both sides
// are HBM, so the kernel is bound by HBM bandwidth and wants the plainest shape
// there is.  One wave moves one tile of 64 vectors (1 KiB at 16-byte vectors)
// and ends; there are as many waves as tiles and the hardware dispatcher deals
// them out, four to a workgroup when packing and one to a workgroup when
// unpacking (scattered stores: 90.6 us against 95.7 for a 256 MiB chunk of 32 KiB
// segments; gathered loads prefer four: 87.8 against 91.4).  No loop, no counters, no second direction;
// loads and stores are non-temporal (nothing is touched twice).  The staging
// side is addressed by list index: segment (plane, i) at
// stage + i * slot_stride + (plane - plane0) * plane_stride.
struct StageParams {
    uint8_t *hbm, *stage;
    uint64_t hbm_plane_stride, hbm_block_stride;
    uint64_t slot_stride, plane_stride;  // staging
    uint32_t plane0, n_planes;           // planes this launch covers
    uint32_t n;                          // blocks
    uint32_t vec_per_seg, tiles_per_seg; // tiles of 64 vectors
    uint32_t tiles;                      // n * n_planes * tiles_per_seg
    uint32_t plane_major;                // tile order: 1 = [plane][i][tile], 0 = [i][plane][tile]
};

template <typename V, bool UNPACK>
__device__ __forceinline__ void stage(const StageParams &p, const int32_t *__restrict__ ids)
{
    const uint32_t lane = threadIdx.x & (kWave - 1u);
    const uint32_t t = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (t >= p.tiles) return;
    const uint32_t segidx = t / p.tiles_per_seg, tin = t - segidx * p.tiles_per_seg;
    uint32_t i, pl;
    if (p.plane_major) {
        pl = segidx / p.n;
        i = segidx - pl * p.n;
    } else {
        i = segidx / p.n_planes;
        pl = segidx - i * p.n_planes;
    }
    const uint32_t v = tin * kWave + lane;
    if (v >= p.vec_per_seg) return;
    V *in_cache = reinterpret_cast<V *>(p.hbm + (uint64_t)(pl + p.plane0) * p.hbm_plane_stride +
                                        (uint64_t)(uint32_t)ids[i] * p.hbm_block_stride) + v;
    V *in_stage = reinterpret_cast<V *>(p.stage + (uint64_t)i * p.slot_stride + (uint64_t)pl * p.plane_stride) + v;
    if constexpr (UNPACK) __builtin_nontemporal_store(__builtin_nontemporal_load(in_stage), in_cache);
    else __builtin_nontemporal_store(__builtin_nontemporal_load(in_cache), in_stage);
}

template <typename V, bool UNPACK>
__global__ __launch_bounds__(kThreads) void kv_stage_kernel(const StageParams p, const int32_t *__restrict__ ids)
{
    stage<V, UNPACK>(p, ids);
}

static_assert(sizeof(StageParams) + sizeof(IdArgs) <= 4096);

template <typename V, bool UNPACK>
__global__ __launch_bounds__(kThreads) void kv_stage_inline_kernel(const StageParams p, const IdArgs a)
{
    stage<V, UNPACK>(p, a.v);
}

// Synthetic decode reader: streams every segment of the named blocks, plane by
// plane (layer-major, as attention over the running requests would), and adds
// up all 32-bit words modulo 2^64.  HBM-bound; read-only.
//
// The bytes to read are one flat sequence of 16-byte vectors, [plane][block][vector],
// cut into tiles of kReadRows rows of 64 vectors (32 KiB, 8 KiB per wave), so a
// tile is full whatever the segment size.  (Tiles that ended with their segment
// read 1500 blocks of 64 x 4 KiB in 243 us, 1/8 of each tile used; the pass alone takes
// 63 us = 6.2 TB/s now, a call with its launch and its wait 79.)
//
// A wave has kReadDepth rows in flight.  One is right: 22 waves per CU with a row
// each are 5.6 MiB over the chip, which is the HBM rate times its latency.  More
// only queue in front of HBM, and a copy over the link that runs beside the
// reader stands in the same queues: 37.5 GiB with 1, 2, 8 rows in flight, TB/s
// alone 7.05, 7.09, 6.99, and GB/s of a rotation beside them 101.1, 89.0, 54.3,
// of a swap-out 56.5, 40.9, 24.0.
//
// Short passes (up to kReadShortRows rows for each wave of the whole grid, 66 MiB) are latency and
// nothing else: tiles of eight rows left most of the grid idle (2 MiB: 64 workgroups, eight
// latencies one behind the other) or half of it in the second of two rounds.  Their tiles are
// as many rows as give every wave about as much, and two rows are in flight.  (As much where a
// wave has 2, 4, 6, 8 or 12 rows: others are rounded up to pairs, so that with one row a wave half of the
// grid has none, and of nine to eleven the second round of six is not full.)  us alone / beside a
// swap-out / a rotation, each with its GB/s, one pass behind the other, before and now:
//    2 MiB  6.8 / 14.9, 57.1 / 22.0, 98.4 and  6.0 /  9.6, 57.1 / 13.9, 95.9
//   28 MiB 11.5 / 17.2, 57.1 / 24.4, 98.2 and 10.5 / 14.5, 57.0 / 19.7, 97.4
//   46 MiB 14.7 / 22.2, 57.0 / 32.6, 99.2 and 13.1 / 16.7, 56.9 / 23.3, 98.1
//   64 MiB 16.6 / 24.0, 57.0 / 34.8, 99.2 and 16.0 / 19.6, 55.4 / 25.4, 97.9
// What the copy loses goes by the number of launches beside it, each of which ends with the caches
// written back, and from 28 MiB on by the second row, too: with one, 64 MiB took 17.7 / 23.5, 57.0 / 31.6, 99.0.
// From 80 MiB on a pass alone gains nothing by it.
//
// No two workgroups meet on an address while they read.  An atomic on one address
// is served every ~14 ns: one counter for the tiles limits claims to 2.3 TB/s per
// 32 KiB, and one sum for all waves (5632 atomics) ended every pass with ~80 us
// of waiting.  So the tiles of a pass are claimed from kReadGroups counters, and
// each workgroup leaves its sum in a place of its own.
struct ReadParams {
    const uint8_t *hbm;
    unsigned long long *part;    // one sum per workgroup, in device memory, from pass to pass
    // Pinned host memory: where the last pass leaves them, each with the device's clock when
    // its workgroup was done, and (nullptr: nowhere) when each of the first kReadBegins began.
    u64x2 *result;
    unsigned long long *begin;
    uint64_t hbm_block_stride;
    uint64_t hbm_plane_stride;
    uint64_t n_vecs;         // n * n_planes * vec_per_seg
    uint64_t seg_magic;      // ceil(2^64 / vec_per_seg) where that divides every n_vecs' index exactly, else 0
    uint32_t n;              // blocks
    uint32_t vec_per_seg;    // seg_bytes / 16
    uint32_t tiles;
    uint32_t rows;           // rows per wave and tile, at most kReadU; a short pass's are even
    uint32_t fixed;          // tiles each workgroup takes without asking (see kv_reader_kernel)
    uint32_t pass, passes;   // pass 0: part[] holds nothing yet
    uint32_t steal;          // groups besides its own that a workgroup takes tiles from
    // Two sets of kReadGroups counters of claimed tiles, kReadStride apart: this pass draws
    // from one, which is zero, and puts the other, the pass before drew from, to zero for
    // the pass behind it.  (Passes on a stream run one after the other.)
    unsigned int *next, *clear;
};

constexpr int kReadU = 8;      // rows per wave and tile
constexpr int kReadDepth = 1;  // rows in flight per wave
constexpr int kReadShortDepth = 2;  // the same in a short pass
constexpr uint32_t kReadShortRows = 12;
constexpr uint32_t kReadRows = (uint32_t)kReadU * (kThreads / kWave);  // rows per tile
constexpr uint32_t kReadVecs = kReadRows * kWave;                      // vectors per tile
constexpr uint32_t kReadBegins = 8;  // workgroups that leave when they began: the first on each XCD
// Counters, and the workgroups that share one: one of every 64 that follow one another,
// each time one place further, so that a group lies on all XCDs and all over each, and
// a copy beside the pass slows every group alike.  37.5 GiB alone / beside a swap-out (whose
// stores went through the L2) and 2 GiB beside it, TB/s: so placed 7.02 / 6.39, 5.88; groups of 22 that follow one another,
// that is on the same three CUs of every XCD, 6.73 / 6.10, 3.55; every 64th workgroup,
// all of a group on one XCD, 6.92 / 5.94, 2.11.  Fewer groups meet more often on their
// counter: 16 read 6.78 alone, 8 6.51.
constexpr uint32_t kReadGroups = 64;
constexpr uint32_t kReadStride = 32;  // 32-bit words from one counter to the next
// A claim is 4 tiles, 2 and at last 1: as long as the group has kReadMargin times as
// many left for each of its workgroups.  A workgroup on a CU with a copy's waves reads
// several times slower than the others and holds two claims, the one it reads and the
// one behind it: they must not outlast the pass.  (8 GiB, TB/s alone / beside a swap-out, as
// above, / a rotation: claims of 1 6.61 / 5.80 / 5.37, of 4 6.81 / 5.94 / 5.38, of 8 6.81 / 5.96 / 5.39;
// claims of 16 with a margin of 2 came to 4.25 beside a swap-out.)
constexpr uint32_t kReadMargin = 16;

// Quotient of a lane's small step past a segment's (or the list's) first entry,
// x < d + 64 * kReadU, without a branch: at d >= 64 * kReadU it is 0 or 1; below,
// the rounded-up reciprocal is exact because x * d < 2^32 (and 1 has none that
// fits, there the quotient is x).
struct SmallDiv {
    uint32_t d, big, magic, one;
    __device__ __forceinline__ explicit SmallDiv(uint32_t div)
        : d(div), big(div >= (uint32_t)(kWave * kReadU) ? div : ~0u),
          magic(div >= (uint32_t)(kWave * kReadU) || div == 1u ? 0u : ~0u / div + 1u), one(div == 1u ? ~0u : 0u)
    {
    }
    __device__ __forceinline__ uint32_t quotient(uint32_t x) const
    {
        return (x >= big ? 1u : 0u) + __umulhi(x, magic) + (x & one);
    }
};

// One wave's share of tile t: kReadU rows (SHORT: p.rows).  ROWS: segments are whole rows, so a
// row has one block id, fetched with a scalar load.  Otherwise rows straddle
// segments and every lane finds its own block and fetches its id itself.  All
// ids are fetched before the first row is.  Past the end of the sequence a row
// (or a lane) repeats the last one that exists, so that no load is conditional,
// and is left out of the sum.  The loads are non-temporal (nothing is read
// twice): worth 16 % on the block-first cache, whose segments lie a whole block apart.
template <bool ROWS, bool SHORT, typename Ids>
__device__ __forceinline__ unsigned long long read_tile(const ReadParams &p, const Ids &ids, uint32_t t, uint32_t wave,
                                                        uint32_t lane)
{
    const uint32_t rows = SHORT ? p.rows : (uint32_t)kReadU;
    const uint32_t row0 = (t * (uint32_t)(kThreads / kWave) + wave) * rows;
    const uint64_t g0 = (uint64_t)row0 * kWave;
    if (g0 >= p.n_vecs) return 0;
    // vectors from this wave's first to the end, as far as they matter here
    const uint32_t left = (uint32_t)min(p.n_vecs - g0, (uint64_t)(rows * kWave));
    const u32x4 *src[kReadU];
    if constexpr (ROWS) {
        const uint32_t rps = p.vec_per_seg / kWave, n_rows = left / kWave;
        const uint32_t segidx = __builtin_amdgcn_readfirstlane(row0 / rps);
        uint32_t pl = __builtin_amdgcn_readfirstlane(segidx / p.n);
        uint32_t r = row0 - segidx * rps, i = segidx - pl * p.n;
        uint32_t word[kReadU], entry[kReadU], plane[kReadU], at[kReadU];
#pragma unroll
        for (uint32_t u = 0; u < (uint32_t)kReadU; u++) {
            if (SHORT && u >= rows) break;
            word[u] = ids.word(i);
            entry[u] = i;
            plane[u] = pl;
            at[u] = r;
            const uint32_t step = u + 1u < n_rows ? 1u : 0u;  // the last row that exists stays
            r += step;
            const uint32_t wrap = r == rps ? 1u : 0u;
            r = wrap ? 0u : r;
            i += wrap;
            const uint32_t next_plane = i == p.n ? 1u : 0u;
            i = next_plane ? 0u : i;
            pl += next_plane;
        }
#pragma unroll
        for (uint32_t u = 0; u < (uint32_t)kReadU; u++) {
            if (SHORT && u >= rows) break;
            src[u] = reinterpret_cast<const u32x4 *>(p.hbm + (uint64_t)plane[u] * p.hbm_plane_stride +
                                                     (uint64_t)ids.id(word[u], entry[u]) * p.hbm_block_stride) + at[u] * kWave + lane;
        }
    } else {
        const uint32_t segidx = (uint32_t)(p.seg_magic ? __umul64hi(g0, p.seg_magic) : g0 / p.vec_per_seg);
        const uint32_t off0 = (uint32_t)(g0 - (uint64_t)segidx * p.vec_per_seg);
        const uint32_t pl0 = __builtin_amdgcn_readfirstlane(segidx / p.n), i0 = segidx - pl0 * p.n;
        const SmallDiv by_seg(p.vec_per_seg), by_list(p.n);
        const uint32_t last = left - 1u;
        uint32_t word[kReadU], entry[kReadU], plane[kReadU], at[kReadU];
#pragma unroll
        for (uint32_t u = 0; u < (uint32_t)kReadU; u++) {
            if (SHORT && u >= rows) break;
            const uint32_t x = off0 + min(u * kWave + lane, last), s = by_seg.quotient(x);
            const uint32_t y = i0 + s, w = by_list.quotient(y);
            entry[u] = y - w * p.n;
            word[u] = ids.word(entry[u]);
            plane[u] = pl0 + w;
            at[u] = x - s * p.vec_per_seg;
        }
#pragma unroll
        for (uint32_t u = 0; u < (uint32_t)kReadU; u++) {
            if (SHORT && u >= rows) break;
            src[u] = reinterpret_cast<const u32x4 *>(p.hbm + (uint64_t)plane[u] * p.hbm_plane_stride +
                                                     (uint64_t)ids.id(word[u], entry[u]) * p.hbm_block_stride) + at[u];
        }
    }
    constexpr int DEPTH = SHORT ? kReadShortDepth : kReadDepth;
    unsigned long long sum = 0;
#pragma unroll
    for (uint32_t u0 = 0; u0 < (uint32_t)kReadU; u0 += DEPTH) {
        if (SHORT && u0 >= rows) break;
        u32x4 v[DEPTH];
#pragma unroll
        for (int k = 0; k < DEPTH; k++) v[k] = __builtin_nontemporal_load(src[u0 + k]);
#pragma unroll
        for (int k = 0; k < DEPTH; k++) {
            const unsigned long long s = (unsigned long long)v[k].x + v[k].y + (unsigned long long)v[k].z + v[k].w;
            sum += (u0 + k) * kWave + lane < left ? s : 0ull;
        }
        asm volatile("" : "+v"(sum));  // the next loads are not issued before these have arrived
    }
    return sum;
}

template <bool ROWS, bool SHORT, typename Ids>
__device__ __forceinline__ void read_pass(const ReadParams &p, const Ids &ids)
{
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1u);
    if (p.begin && blockIdx.x < kReadBegins && tid == 0)
        __scoped_atomic_store_n(p.begin + blockIdx.x, (unsigned long long)wall_clock64(), __ATOMIC_RELAXED, __MEMORY_SCOPE_SYSTEM);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    __shared__ uint32_t claimed[2];
    __shared__ unsigned long long sums[kThreads / kWave];
    // first the fixed share, a tile every gridDim.x ...
    const uint32_t n_fixed = (uint32_t)min((uint64_t)p.fixed * gridDim.x, (uint64_t)p.tiles);
    // ... then tiles n_fixed + group + n_groups * c, c drawn from the group's counter, and
    // once the group has none left, from those of the next p.steal groups
    const uint32_t n_groups = min(gridDim.x, kReadGroups), per_group = (gridDim.x + n_groups - 1u) / n_groups;
    const uint32_t shared = p.tiles - n_fixed, each = shared / n_groups, extra = shared - each * n_groups;
    uint32_t group = (blockIdx.x + blockIdx.x / kReadGroups) % n_groups, steals = min(p.steal, n_groups - 1u);
    uint32_t size = each + (group < extra ? 1u : 0u);  // tiles of the group
    auto claim_size = [&](uint32_t c) {  // tiles of the claim that follows tile c of the group
        const uint32_t left = size - min(c, size), round = kReadMargin * per_group;
        return left > 4u * round ? 4u : left > 2u * round ? 2u : 1u;
    };
    // the next claim is always in flight while the tiles before it are read
    uint32_t pending = 0, want = claim_size(0);
    if (shared && tid == 0) pending = atomicAdd(p.next + group * kReadStride, want);
    unsigned long long sum = 0;
    uint32_t t = blockIdx.x, end = n_fixed, step = gridDim.x;
    for (uint32_t turn = 0;; turn ^= 1u) {
        for (; t < end; t += step) sum += read_tile<ROWS, SHORT>(p, ids, t, wave, lane);
        if (!shared) break;
        if (tid == 0) claimed[turn] = pending;
        __syncthreads();  // one per claim: the two slots alternate
        const uint32_t c = __builtin_amdgcn_readfirstlane(claimed[turn]);
        if (c >= size) {
            if (steals == 0) break;
            steals--;
            group = group + 1u == n_groups ? 0u : group + 1u;
            size = each + (group < extra ? 1u : 0u);
            want = 1u;
        } else {
            step = n_groups;
            t = n_fixed + group + n_groups * c;
            end = n_fixed + group + n_groups * min(c + want, size);
            want = claim_size(c + want);
        }
        if (tid == 0) pending = atomicAdd(p.next + group * kReadStride, want);
    }
    if (blockIdx.x == gridDim.x - 1u && tid < kReadGroups) p.clear[tid * kReadStride] = 0u;
    // one sum per workgroup, in a place of its own (the host adds them up)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    if (lane == 0) sums[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kThreads / kWave; w++) sum += sums[w];
        if (p.pass > 0) sum += p.part[blockIdx.x];
        const unsigned long long now = wall_clock64();
        if (p.pass + 1u < p.passes) p.part[blockIdx.x] = sum;
        else store_host<u32x4, true>(__builtin_bit_cast(u32x4, u64x2{sum, now}), reinterpret_cast<u32x4 *>(p.result + blockIdx.x));
    }
}

template <bool ROWS, bool SHORT>
__global__ __launch_bounds__(kThreads) void kv_reader_kernel(const ReadParams p, const int32_t *__restrict__ ids)
{
    read_pass<ROWS, SHORT>(p, IdsInMemory{ids});
}

template <bool ROWS, bool SHORT, typename Ids>
__global__ __launch_bounds__(kThreads) void kv_reader_inline_kernel(const ReadParams p, const IdArgs a)
{
    read_pass<ROWS, SHORT>(p, Ids{a});
}

static_assert(sizeof(ReadParams) + sizeof(IdArgs) <= 4096);

// Before the passes of a list that arguments do not hold: from pinned host memory to the
// device.  (A list of 1500 blocks of 64 x 4 KiB was read in 85 us with it, and is in 81
// without.)
__global__ __launch_bounds__(kThreads) void kv_reader_ids_kernel(const int32_t *__restrict__ from, int32_t *__restrict__ ids,
                                                                 uint32_t n)
{
    for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) ids[i] = from[i];
}

}  // namespace dkv
