// hv_kernels.h -- launchers shared between the kernel sources and the C ABI.
// Every launcher queues work on `stream` and returns the launch status; it
// trusts its arguments (the C ABI validates them first).
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <hip/hip_runtime.h>

namespace hv {

// Hash algorithm of a call: SHA-256 (32-byte digests, 64-byte blocks) or
// SHA-384 (48-byte digests, 128-byte blocks).
constexpr int kAlgSha256 = 0;
constexpr int kAlgSha384 = 1;

// One leaf as the hash kernel sees it.
struct LeafDesc {
    uint64_t src;     // device address of the chunk's first byte
    uint64_t nbytes;  // chunk length in bytes
    uint64_t out;     // leaf index: the digest goes to leaf_digests + 32 * out
};

// Message descriptor as uploaded (same layout as hv_msg).
struct MsgDesc {
    uint64_t data;
    uint64_t nbytes;
};

// Scratch of a balanced leaf launch (balance.h): the table's work as one tape,
// cut into an interval per wave.  All pointers are device memory.
struct Tape {
    uint64_t* head;     // full groups, then the tape position of every other group of 64 slots, and its end
    uint32_t* ready;    // per wave: its saved states may be read
    uint8_t* states;    // per wave: kTapeStateBytes
    uint64_t full_len;  // length on the tape of a group of full chunks
    uint32_t setup;     // part of every group's length before its blocks
    uint32_t waves;     // a multiple of 4
    uint32_t polls;     // looks for the states of the wave before
};
// What a group costs a wave besides its blocks, in blocks: its descriptors, the
// first stage's loads, the final block and the digests take some 7 us (SHA-256)
// to 12, and a tape has no fourth wave on a SIMD to hide them.  Without them an
// interval of short tails took far longer than the others: 70,000 chunks of
// 4 KiB, a fourth of them tails of 100 bytes, 279 us against 184 with the plain
// launch, 188 with them; SHA-384, the tails of every length, 288 and 207, 216.
// Where nearly all chunks are whole ones they change nothing (205,697 of 64 KiB:
// 7.81 ms without, 7.80 with them).
constexpr uint32_t kTapeSetup256 = 3, kTapeSetup384 = 2;
// Looks of a wave that waits for another's states, at least; for chunks of more
// blocks than that, one for each block, which is still less than the time they
// take to hash again (a look is 0.4 us and more, a block 2.6 and more).
constexpr uint32_t kTapePolls = 1 << 14;
constexpr uint64_t kTapeStateBytes = 64 * 64;
constexpr uint32_t kTapeMaxWaves = 3 * 1024;  // three per SIMD of 256 CUs

// Per-message counts / offsets: x = full chunks, y = tail leaves (0 or 1).
using Pair = ulonglong2;

constexpr int kSortBuckets = 4096;   // block-count classes of the tail sort

// Leaf launchers split a call into launches of at most this many leaf-table
// slots, so a grid stays below a dispatch's 2^32 work-items at two lanes per
// slot (the chain kernels).
constexpr uint64_t kMaxSlotsPerLaunch = (uint64_t)1 << 30;

// Scheduler (sched.hip).
hipError_t launch_fill_u64(uint64_t* p, size_t n, uint64_t v, hipStream_t s);
// Copies a host table of n words to the device; `from` is read before the call
// returns.  A pageable copy waits for the stream and is waited for, so the
// kernels behind it start some 20 us after the ones before it end; tables of up
// to 15 KB (30 KB where every word fits 32 bits) go as launch arguments
// instead, at most four launches of about 4 us: a one-shot call over 24 short
// tensors 163 -> 138 us, over 720 222 -> 204; rehashing 1000 chunks and updating
// the tree above them, its table behind the leaf kernel in the stream, 1.47 ->
// 1.43 ms.  Four launches on an idle stream take as long as the copy, and with
// more the copy is faster: leaf digests of 1,025 messages 115 us with five
// launches and 107 with the copy, a tree update of 5,760 leaves 219 and 188.  A
// stream under capture gets the copy whatever the size.
hipError_t upload_table(uint64_t* to, const uint64_t* from, size_t n, hipStream_t s);
hipError_t launch_sched_count(const MsgDesc* msgs, uint32_t n, uint64_t C, Pair* cnt, hipStream_t s);
size_t scan_partials_count(size_t n);
hipError_t launch_scan_pairs(const Pair* in, Pair* out, size_t n, Pair* partials, hipStream_t s);
hipError_t launch_sched_full(const MsgDesc* msgs, const Pair* off, uint32_t n, uint64_t C, uint64_t n_full,
                             LeafDesc* desc, hipStream_t s);
hipError_t launch_sched_tails(const MsgDesc* msgs, const Pair* off, uint32_t n, uint64_t C, uint64_t n_full,
                              uint64_t* hist, LeafDesc* desc, hipStream_t s);

// The same table and offsets in one launch for up to kSmallMessages messages
// (0 < n), and select's.  A one-shot call over 24 short tensors, hash to
// verdict: 285 us with the nine launches, 243 with this one.
constexpr uint32_t kSmallMessages = 1024;
hipError_t launch_sched_small(const MsgDesc* msgs, uint32_t n, uint64_t C, uint64_t n_full, Pair* off, LeafDesc* desc,
                              hipStream_t s);
hipError_t launch_select_small(const MsgDesc* msgs, uint32_t n, uint64_t C, const uint64_t* leaves, uint64_t k,
                               LeafDesc* desc, hipStream_t s);

// Lays a scheduled leaf table (full chunks first, then tails by falling block
// class) out as a tape for t.waves waves and clears t.ready; off[n_msgs].x is
// the number of full chunks.
hipError_t launch_tape_plan(int alg, const LeafDesc* desc, uint64_t n_slots, const Pair* off, uint32_t n_msgs,
                            const Tape& t, hipStream_t s);
// The one-wave leaf kernels over a planned tape.
hipError_t launch_sha256_tape(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              const Tape& t, hipStream_t s);
hipError_t launch_sha384_tape(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              const Tape& t, hipStream_t s);
// Waves of the tape that a one-wave call over n_slots leaves, nearly all of
// them full chunks, is cut into on a device of `cus` compute units; 0 where the
// plain launch is as fast.
uint32_t tape_waves(uint64_t n_slots, uint32_t cus);

// SHA-384 of the n_slots leaves of a leaf table (sha384_leaves.hip): 48-byte
// digests at digests + 48 * desc.out for desc.out < out_bound.
hipError_t launch_sha384_leaves(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                                hipStream_t s);

// Leaf table for a sorted list of leaf numbers (sched.hip): desc[e] is leaf
// leaves[e], located through the per-message offsets `off` (first leaf of
// message m = off[m].x + off[m].y).
hipError_t launch_sched_select(const MsgDesc* msgs, const Pair* off, uint32_t n, uint64_t C, const uint64_t* leaves,
                               uint64_t k, LeafDesc* desc, hipStream_t s);

// SHA-256 of the n_slots leaves of a leaf table (sha256_leaves.hip); digests
// go to digests + 32 * desc.out for desc.out < out_bound.
// Leaf table of leaves [first, first + k) into desc[0..k) (digest slot e for
// leaf first + e); also resets reset[0] = 0, reset[1] = ~0 when reset != NULL.
hipError_t launch_sched_range(const MsgDesc* msgs, const Pair* off, uint32_t n, uint64_t C, uint64_t first,
                              uint64_t k, LeafDesc* desc, uint64_t* reset, hipStream_t s);
// Monitor comparison: for e < k, digest e (D bytes at digests + D*e) against
// reference leaf first + e (ref + D*(first + e)); result[0] += mismatches,
// result[1] = min(result[1], lowest mismatching leaf number).  D is 32 or 48.
hipError_t launch_monitor_compare(const uint8_t* digests, const uint8_t* ref, uint64_t first, uint64_t k, uint32_t D,
                                  uint64_t* result, hipStream_t s);
// The SHA-256 chain kernel (sha256_split.hip; same contract as
// launch_sha256_leaves), with one or two groups of 64 chunks per workgroup.
// The automatic choice takes it for up to 128 leaves per compute unit of the
// current device (32768 on a 256-CU device).
hipError_t launch_sha256_split(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                               bool two_groups, hipStream_t s);
// The SHA-384 chain kernel and, with two_pairs, the kernel of two
// producer/consumer pairs (sha384_split.hip; same contract as
// launch_sha384_leaves).
hipError_t launch_sha384_split(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                               bool two_pairs, hipStream_t s);
// SHA-384 leaf digests with the kernel the choice selects (the callers' entry),
// by the same rules as launch_sha256_auto.
hipError_t launch_sha384_auto(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              hipStream_t s, bool background = false);
// What a leaf launch runs (hv_leaf_launch_for's values).
enum : int {
    kLeafOneWave = 1,
    kLeafTwoWave = 2,         // the chain kernels, 64 chunks per workgroup
    kLeafTwoWaveCompact = 3,  // 128 chunks: SHA-256's chain kernel, SHA-384's two pairs
    kLeafThreeGroup = 4,      // SHA-256 only
    kLeafTape = 5,            // one-wave over a tape (Tape)
};
// The kernel a launch over n_slots leaves takes under this thread's choice on
// a device of `cus` compute units, where it has no tape.
int leaf_launch_for(int alg, uint64_t n_slots, bool background, uint64_t cus);
// Compute units of the current device (queried once per device; 0 if the
// query fails, which makes the automatic choices take the one-wave kernels).
uint32_t device_cus();
// Leaf-kernel choice of the calling thread (hv_set_leaf_kernel): 0 automatic,
// 1 one-wave kernel, 2 the kernels for small leaf counts (launch_sha256_split,
// launch_sha384_split), 3 those with 128 chunks per workgroup.
int leaf_kernel_choice();
// SHA-256 leaf digests with the kernel that choice selects (the callers' entry).
// background: work that shares the chip with other work (monitor scans);
// under the automatic choice it takes the one-wave kernel, which hashes a byte
// with the fewest instructions, rather than the one with the shortest chains.
hipError_t launch_sha256_auto(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              hipStream_t s, bool background = false);
hipError_t launch_sha256_leaves(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                                hipStream_t s);

// Merkle tiles (merkle.hip).  One launch reduces every segment by up to
// kTileLevels levels: tile t covers up to 2^kTileLevels consecutive nodes of
// one segment and writes one node.
constexpr int kTileLevels = 9;
constexpr int kTileNodes = 1 << kTileLevels;
hipError_t launch_merkle_tiles(int alg, const uint8_t* in, uint8_t* out, const uint64_t* in_off,
                               const uint64_t* tile_off, uint32_t n_seg, uint64_t n_tiles, int leaf_mode,
                               hipStream_t s);
// Merkle groups (merkle.hip), the launches over the widest levels: group g
// -- up to 2^kGroupLevels consecutive nodes of one segment, starting at a
// multiple of that -- is reduced to one node in registers, by one lane for
// g < n_main and by four lanes (two entries each, then two shuffle levels)
// for the launch's last groups, g >= n_main.
constexpr int kGroupLevels = 3;
constexpr int kGroupNodes = 1 << kGroupLevels;
constexpr int kGroupQuad = 4;  // lanes per group beyond n_main
hipError_t launch_merkle_groups(int alg, const uint8_t* in, uint8_t* out, const uint64_t* in_off,
                                const uint64_t* grp_off, uint32_t n_seg, uint64_t n_groups, uint64_t n_main,
                                int leaf_mode, hipStream_t s);

// Persistent tree for incremental updates (tree.hip).
hipError_t launch_tree_leaf_level(int alg, const uint8_t* digests, uint64_t n, uint8_t* level0, hipStream_t s);
hipError_t launch_tree_build_level(int alg, const uint8_t* in, uint8_t* out, const uint64_t* in_off,
                                   const uint64_t* out_off, uint32_t n_seg, uint64_t n_out, hipStream_t s);
hipError_t launch_tree_locate(const uint64_t* dirty, uint32_t k, const uint64_t* seg_off, uint32_t n_seg,
                              uint32_t* seg_of, uint64_t* local, hipStream_t s);
hipError_t launch_tree_update_leaves(int alg, const uint8_t* digests, const uint64_t* dirty, uint32_t k,
                                     uint8_t* level0, hipStream_t s);
hipError_t launch_tree_update_level(int alg, const uint8_t* in, uint8_t* out, const uint64_t* in_off,
                                    const uint64_t* out_off, const uint32_t* seg_of, const uint64_t* local, uint32_t k,
                                    uint32_t shift, hipStream_t s);
hipError_t launch_tree_roots(int alg, const uint8_t* top, const uint64_t* top_off, uint32_t n_seg, uint8_t* roots,
                             hipStream_t s);

// Verification (verify.hip).
// nbytes: 32 or 48 (the digest size of the call's hash).
hipError_t launch_verify_root(const uint8_t* root, const uint8_t* expected, uint32_t nbytes, uint32_t* flag,
                              hipStream_t s);
// As launch_verify_root with `expected` (nbytes) in device memory.
hipError_t launch_verify_root_dev(const uint8_t* root, const uint8_t* expected, uint32_t nbytes, uint32_t* flag,
                                  hipStream_t s);
hipError_t launch_compare_roots(const uint8_t* roots, const uint8_t* expected, uint32_t n, uint32_t nbytes,
                                uint32_t* mismatch, hipStream_t s);

}  // namespace hv
