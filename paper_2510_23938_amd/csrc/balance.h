// balance.h -- an even split of a leaf table's work over the waves of a
// one-wave leaf kernel, chunks cut between waves where that makes it even.
//
// One wave hashes 64 chunks, and the chip runs whole waves: 205,697 chunks of
// 64 KiB are 3.14 waves per SIMD, which run as three at once and then a fourth
// nearly alone (10.5 ms; 7.8 is the work's share, and 8.1 what a tape takes,
// SHA-384 13.3 and 10.1; 66,000 chunks: 5.1 and 2.8 ms).  A chunk is a chain,
// but a chain can be cut: its state after some block is 32 or 64 bytes, and
// another wave can go on from it.  So the table's groups of 64 slots are laid
// end to end on a tape (a group's length: its set-up and its most blocks), the tape is cut
// into one equal interval per resident wave, and a group across a boundary is
// shared by the two intervals (the wrap-around rule of preemptive scheduling
// on identical machines, McNaughton 1959): the interval on the right hashes
// the group's first blocks at its start and saves the states, the one on the
// left goes on from them at its end.  An interval is at least as long as the
// longest group, so no group meets more than two intervals, and the first
// part, at the start of its interval, is done before the second is due.
//
// Wave k takes the k-th interval from the right, so a wave only ever waits
// for the wave before it, which was dispatched no later.  The wait is bounded
// all the same: a wave that does not see the states in time hashes the group
// from its first block, with the same result (load_states).
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

#include "hv_kernels.h"

namespace hv {

constexpr uint64_t kStateBytes = kTapeStateBytes;  // 64 lanes of at most eight 64-bit words

// One stretch of a wave's interval: blocks [from, to) of group `group`.
struct Piece {
    uint64_t group;
    uint32_t from, to;  // from > 0: go on from the states of the wave before
    bool last;          // to is the group's end (padding included); else, to is 0
                        // where only set-up lies in this interval
};

// The intervals of a tape, walked by one wave: all values are wave-uniform.
struct TapeWalk {
    const uint64_t* tail_start;  // tape position of each group with a tail, and the tape's end
    uint64_t full_groups;        // the groups of full chunks only, the table's first
    uint64_t full_len;           // length of each of them
    uint32_t setup;              // of a group's length, before its blocks
    uint64_t group, start;       // the group `pos` lies in, and its tape position
    uint64_t pos, end;           // what is left of the interval

    __host__ __device__ __forceinline__ TapeWalk(const Tape& t, uint64_t n_slots, uint32_t wave)
        : tail_start(t.head + 1), full_groups(t.head[0]), full_len(t.full_len), setup(t.setup) {
        const uint32_t tail_groups = (uint32_t)((n_slots + 63) / 64 - full_groups);
        const uint64_t total = tail_start[tail_groups];
        uint64_t share = (total + t.waves - 1) / t.waves;
        // the longest group is a full one or the first of the others (theirs
        // are class bounds, not rising)
        const uint64_t other = tail_groups > 0 ? tail_start[1] - tail_start[0] : 0;
        const uint64_t longest = full_groups > 0 && full_len > other ? full_len : other;
        share = share > longest ? share : longest;
        pos = share * (t.waves - 1 - wave);
        end = pos + share < total ? pos + share : total;
        if (pos < full_groups * full_len) {
            group = pos / full_len;
            start = group * full_len;
        } else {
            uint32_t lo = 0, hi = tail_groups;  // tail_start[lo] <= pos < tail_start[hi], or pos >= end
            while (hi > lo + 1) {
                const uint32_t mid = lo + (hi - lo) / 2;
                if (tail_start[mid] <= pos) lo = mid; else hi = mid;
            }
            group = full_groups + lo;
            start = tail_start[lo];
        }
    }

    __host__ __device__ __forceinline__ bool next(Piece* p) {
        if (pos >= end) return false;
        const uint64_t len =
            group < full_groups ? full_len : tail_start[group - full_groups + 1] - tail_start[group - full_groups];
        const uint64_t left = pos - start;                                 // of the group, in the interval before
        const uint64_t here = start + len < end ? len - left : end - pos;  // of the group, in this one
        p->group = group;
        // at the interval's start the group's first blocks; at its end the last ones
        p->last = left == 0;
        const uint32_t from = p->last ? (uint32_t)(len - here) : 0u, to = from + (uint32_t)here;
        // a cut lies on an even block: two SHA-256 blocks are a stage and a
        // 128-byte line, and from an odd one on every stage would be of two lines
        p->from = from > setup ? (from - setup) & ~1u : 0u;
        p->to = p->last ? to - setup : to > setup ? (to - setup) & ~1u : 0u;
        pos += here;
        start += len;
        ++group;
        return true;
    }
};

// Saves this wave's chunk states (NW 32-bit words per lane) and says so.
template <int NW>
__device__ __forceinline__ void save_states(const Tape& t, uint32_t wave, const uint32_t* s) {
    uint32_t* to = reinterpret_cast<uint32_t*>(t.states + kStateBytes * wave) + (threadIdx.x & 63);
#pragma unroll
    for (int i = 0; i < NW; ++i) to[64 * i] = s[i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_store(t.ready + wave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The states the wave before saved; false when they do not come in time: after
// t.polls looks, 0.4 us apart and more.
template <int NW>
__device__ __forceinline__ bool load_states(const Tape& t, uint32_t wave, uint32_t* s) {
    bool there = false;
    for (uint32_t tries = 0; tries < t.polls && !there; ++tries) {
        there = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(t.ready + (wave - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0;
        if (!there) __builtin_amdgcn_s_sleep(16);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (!there) return false;
    const uint32_t* from = reinterpret_cast<const uint32_t*>(t.states + kStateBytes * (wave - 1)) + (threadIdx.x & 63);
#pragma unroll
    for (int i = 0; i < NW; ++i) s[i] = from[64 * i];
    return true;
}

}  // namespace hv
