// hv_host.h -- host-side internals shared by the C-ABI sources: argument
// errors, workspace carving and the scheduling launch sequence.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "hv.h"
#include "hv_kernels.h"

namespace hvh {

constexpr size_t kAlign = 256;
inline size_t round_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Largest leaf (or tree entry) count one call accepts.  It keeps the kernels'
// 32-bit grid-stride indices below 2^32 and is far above what fits in HBM
// (every leaf takes a 24-byte table entry and its digest besides its bytes).
constexpr uint64_t kMaxLeaves = (uint64_t)1 << 31;
// Largest chunk: the leaf kernels count a chunk's 64-byte blocks, padding
// blocks included, in 32 bits; 2^31 whole blocks leave room for the padding
// and for the kernels' rounding of block counts to pairs.
constexpr uint64_t kMaxChunkBytes = (uint64_t)1 << 37;

// Carves consecutive 256-byte-aligned regions out of a workspace.
struct Carver {
    uint8_t* base;
    size_t used = 0;
    explicit Carver(void* b) : base(static_cast<uint8_t*>(b)) {}
    template <typename T>
    T* take(size_t count) {
        T* p = reinterpret_cast<T*>(base ? base + used : nullptr);
        used += round_up(count * sizeof(T));
        return p;
    }
};

struct HashLayout {
    hv::MsgDesc* msgs;
    hv::Pair* cnt;
    hv::Pair* off;
    hv::Pair* partials;
    uint64_t* hist;
    hv::LeafDesc* desc;
    size_t bytes;
    // beyond `bytes`, where a balanced leaf launch may pay (tape_worth): its
    // scratch.  tape_bytes is the end of it (`bytes` where there is none); a
    // workspace that ends sooner is enough, and the plain launch runs.
    hv::Tape tape;
    size_t tape_bytes;
};

HashLayout hash_layout(void* ws, uint32_t n_msgs, uint64_t n_leaves);

// Calls for which the leaf table's work may be split evenly over the resident
// waves (balance.h), and which have scratch for it: more than one wave per SIMD
// (256 CUs), up to 8 (beyond that a partly filled last round is a few percent,
// no more than the walk costs: 700,000 and 10^6 chunks took 0.98 to 1.00 of the
// plain launch's rate), and few messages per leaf, so that nearly all chunks are
// full ones when the call has a chunk size at all.
inline bool tape_worth(uint32_t n_msgs, uint64_t n_leaves) {
    return n_leaves > 65536 && n_leaves <= (1u << 19) && n_msgs <= n_leaves / 4;
}
// Of those, the calls whose chunks are long enough: a tape has three waves on a
// SIMD where the plain launch has four and more for chunks of a few blocks, and
// its plan is a launch of its own.  Tape against plain: 1 KiB chunks 0.8 to 1.1
// from 115,000 leaves on (512-byte ones 0.65 to 0.8), 2 KiB 1.0 to 1.5 where few
// are tails and 0.86 to 1.3 where a seventh are, 4 KiB 0.96 to 1.6, 64 KiB 1.0 to
// 1.8.
inline bool tape_chunks(uint32_t n_msgs, uint64_t n_leaves, uint64_t chunk_bytes) {
    return chunk_bytes >= 4096 || (chunk_bytes >= 2048 && n_msgs <= n_leaves / 16);
}

// A message table to the device; `msgs` is read before the call returns.
inline hipError_t upload_messages(hv::MsgDesc* to, const hv_msg* msgs, uint32_t n_msgs, hipStream_t stream) {
    static_assert(sizeof(hv_msg) == 2 * sizeof(uint64_t) && sizeof(hv::MsgDesc) == sizeof(hv_msg), "message layout");
    return hv::upload_table(reinterpret_cast<uint64_t*>(to), reinterpret_cast<const uint64_t*>(msgs),
                            2 * (size_t)n_msgs, stream);
}

// What launch_leaves runs for such a table on a device of `cus` compute units
// under this thread's choice (hv::kLeaf...), with the tape's scratch; for
// kLeafTape, *waves is the tape's.
int leaf_launch(hv_alg alg, uint32_t n_msgs, uint64_t chunk_bytes, uint64_t n_leaves, uint32_t cus, uint32_t* waves);

// The leaf kernel of a scheduled table (L.desc, L.off): the automatic choice,
// over a tape where `tape` (L's tape scratch is there) and it pays.
hipError_t launch_leaves(hv_alg alg, const HashLayout& L, bool tape, uint32_t n_msgs, uint64_t chunk_bytes,
                         uint64_t n_leaves, uint8_t* digests, hipStream_t stream);

// Records a detail string for hv_last_error() and returns st.
hv_status fail(hv_status st, const char* fmt, ...);
hv_status hip_fail(hipError_t e, const char* what);

// Leaf counts of a message list (validation included); fills seg_offsets when given.
hv_status layout(const hv_msg* msgs, uint32_t n_msgs, uint64_t C, uint64_t* seg_offsets, uint64_t* n_leaves,
                 uint64_t* n_full);

// The body of hv_hash_chunks_alg over a given workspace (validation, descriptor
// upload, scheduling, leaf kernel).  With `events` the call may create and use
// HIP events: a large descriptor table is then uploaded asynchronously while
// the host validates it, and the leaf kernel is timed when
// hv_set_kernel_timing is on; without, it creates no runtime object.
hv_status hash_chunks_into(hv_alg alg, const hv_msg* msgs, uint32_t n_msgs, uint64_t chunk_bytes,
                           uint8_t* leaf_digests, void* workspace, size_t workspace_bytes, bool events,
                           hipStream_t stream);

// Scheduling kernels over device-resident descriptors into L (leaf table in L.desc).
hv_status queue_schedule(const hv::MsgDesc* msgs_dev, uint32_t n_msgs, uint64_t chunk_bytes, uint64_t n_full,
                         uint64_t n_leaves, const HashLayout& L, hipStream_t stream);

// Segmented Merkle reductions chain launches, each a group launch (3 levels in
// registers, one or four lanes per group of 8 entries) or a tile launch (9
// levels, a workgroup per 512-node tile).  Launch k (from 1) over `entries`
// nodes in n_seg segments is a group launch
//   - from kGroupMinNodes entries on, where the widest levels keep every lane
//     busy, or
//   - for more than kManySegments segments of at most 8 entries on average,
//     where one to three group launches save a tile launch (merkle_short_groups):
//     a tile is a workgroup however few nodes it has, three at a time on a CU,
//     and reduces them at one wave's latency (20,000 segments of 1 to 13
//     entries: 886 us), while a group is a lane or four (two launches, see
//     merkle_group_main: 40 us).
// Up to 2^31 entries (the per-call limit) that is at most 5 group launches and
// 2 tile launches; with launches of the second kind, which start below
// kGroupMinNodes entries, at most 6 in all.
constexpr int kMaxMerkleLaunches = 8;
constexpr uint64_t kGroupMinNodes = (uint64_t)1 << 18;
constexpr uint32_t kManySegments = 1536;  // two rounds of tiles on 256 CUs
// Tile launches that reduce a segment of c nodes to one.
inline int merkle_tile_launches(uint64_t c) {
    int t = 0;
    for (; c > 1; ++t) c = (c + hv::kTileNodes - 1) / hv::kTileNodes;
    return t;
}
// Whether launch k may be a group launch of the second kind, and is asked next.
inline bool merkle_many_short(uint64_t entries, uint32_t n_seg, int k) {
    return k <= 3 && n_seg > kManySegments && entries <= 8 * (uint64_t)n_seg && entries < kGroupMinNodes;
}
// The group launches, from launch k on, that save a tile launch of a reduction
// with `entries` nodes left, at most `longest` in a segment (that, or the next
// power of two); 0 for a tile launch.  A launch that saves none is time lost
// (20,000 segments and one of 300,000 entries: 0.97 ms, 1.09 with two more group
// launches; planning and sending one takes 5 ns a segment, where a tile takes 20
// even with a single node), unless the tiles have much to hash, four nodes each
// (40 entries and then 5 each: 1.16 ms, 0.97).  And for up to twice
// kManySegments only where it saves them all, in two launches at most (one after
// the first), and not where the tiles are quick, two SHA-384 entries at most: 2,000 segments of up to two
// entries 98 us with the tile launch, 110 with the group launch; with one of 500
// among them 101 and 119 (SHA-256), 125 and 168, of 12,000 171 and 192; 5,000
// 171 and 102, 174 and 131, 171 and 174, 270 and 233.
inline int merkle_short_groups(uint64_t entries, uint64_t longest, uint32_t n_seg, int k, bool sha384) {
    const int tiles = merkle_tile_launches(longest) + (k == 1 && longest <= 1 ? 1 : 0);
    const bool more = n_seg > 2 * kManySegments;
    if (sha384 && longest <= 2 && !more) return 0;
    uint64_t c = longest;
    for (int j = 1; j <= 4 - k; ++j) {
        c = (c + hv::kGroupNodes - 1) / hv::kGroupNodes;
        if (more ? merkle_tile_launches(c) < tiles : c <= 1 && j <= (k == 1 ? 2 : 1)) return j;
    }
    return more && entries >= 4 * (uint64_t)n_seg ? 1 : 0;
}

// Host plan of a segmented Merkle reduction over validated segment offsets:
// `table` gets rows of n_seg + 1 offsets -- row 0 the segment offsets, row k
// the first output node of each segment after launch k (a segment with c
// nodes gets max(1, ceil(c / w)) outputs, w = 8 for a group launch and 512 for
// a tile launch) -- `launches` the launch count and bit k - 1 of `groups` is set
// where launch k is a group launch of the second kind above.
hv_status merkle_plan(const uint64_t* seg_offsets, uint32_t n_seg, bool sha384, std::vector<uint64_t>* table,
                      int* launches, uint32_t* groups);
inline bool merkle_grouped(uint64_t entries, uint32_t groups, int k) {
    return entries >= kGroupMinNodes || ((groups >> (k - 1)) & 1u) != 0;
}

// Segment offsets: start at 0, never decrease, at most the per-call entry limit.
hv_status check_segments(const uint64_t* seg_offsets, uint32_t n_seg);

// The launches a reduction of these (checked) segments makes on a device of
// `cus` compute units (hv_merkle_launches in hv_inspect.h).
hv_status merkle_launch_kinds(hv_alg alg, const uint64_t* seg_offsets, uint32_t n_seg, uint32_t cus, int* launches,
                              int* kind, uint64_t* units, uint64_t* one_lane);

// Groups a group launch of n_groups groups gives one lane each (the rest, its
// last groups, get four lanes each), for a device of `cus` compute units
// (4 SIMDs each).  A wave of one-lane groups takes D block times (8 entries:
// the leaf hashes in leaf mode, then 7 nodes), a wave of four-lane groups d
// (2 entries, then 3 nodes along the chain) for a quarter of the groups.
// With R = 256 * cus groups per wave on every SIMD, all one-lane costs
// ceil(G / R) * D on the busiest SIMD; the split keeps floor(G / R) whole
// rounds and spreads the rest as four-lane waves, k * D + ceil(4r / R) * d.
// The split is taken when it costs less: it shortens the launch's last round,
// where one wave per SIMD would otherwise run alone.  A launch of less than a
// round is all four-lane for many short segments (there is nothing else on the
// chip) and all one-lane from kGroupMinNodes entries on.
inline uint64_t merkle_group_main(uint64_t n_groups, uint64_t entries, bool leaf_mode, bool sha384, uint32_t cus) {
    if (cus == 0) return n_groups;
    const uint64_t leaf = leaf_mode ? 1 : 0, node = sha384 ? 1 : 2;  // 64- or 128-byte blocks per hash
    const uint64_t D = 8 * leaf + 7 * node, d = 2 * leaf + 3 * node;
    const uint64_t R = 256 * (uint64_t)cus;
    const uint64_t k = n_groups / R, r = n_groups % R;
    if (r == 0 || (k == 0 && entries >= kGroupMinNodes)) return n_groups;
    const uint64_t all = (k + 1) * D, split = k * D + (4 * r + R - 1) / R * d;
    return split < all ? k * R : n_groups;
}

// Nodes any launch of a reduction of n_nodes nodes in n_seg segments writes, at most.
uint64_t merkle_tiles_bound(uint64_t n_nodes, uint32_t n_seg);

// Queues the launches of a planned reduction: `in` (entries; the first launch
// forms their leaf hashes) through ping / pong into `out`.  table: the plan's
// rows on the device; outputs[k]: nodes written by launch k + 1; groups: the plan's.
hv_status queue_merkle(hv_alg alg, const uint8_t* in, uint8_t* out, const uint64_t* table, uint32_t n_seg,
                       uint64_t n_nodes, int launches, const uint64_t* outputs, uint32_t groups, uint8_t* ping,
                       uint8_t* pong, hipStream_t stream);

// HIP events around a leaf kernel on `stream` when hv_set_kernel_timing is on
// for this thread (no-ops otherwise).
hv_status leaf_timing_start(hipStream_t stream);
hv_status leaf_timing_stop(hipStream_t stream);

}  // namespace hvh
