// sha256_split.hip -- SHA-256 of every chunk for small leaf counts: two lanes
// per chunk and a schedule made by other waves, so that one chunk's chain of
// blocks runs faster.
//
// With fewer chunks than the chip has lanes, a chunk's time is the latency of
// its chain of compressions, and a lone wave issues one VALU instruction every
// 4.6 to 4.8 cycles whatever its operands: what bounds a block is the number
// of instructions on the wave that carries the state.  The one-wave kernel has
// 1405 of them per block.  Two things take instructions off that wave:
//
// 1. Producer waves build each block's 64 schedule words -- message words,
//    padding (section 5.1.1) and expansion (FIPS 180-4 section 6.2.2 step 1),
//    each with its round constant added -- into LDS; consumer waves only run
//    rounds.
// 2. A chunk has two lanes of a consumer wave.  The a lane holds the last four
//    values of a (a, b, c, d of the round), the e lane those of e (e, f, g, h):
//      e' = Sigma1(e) + Ch(e, f, g) + (h + K + W) + d
//      a' = Sigma0(a) + Maj(a, b, c) + e' - d
//    Both are sigma(x0) + f(x0, x1, x2) +- x3 + one value of the partner's, so
//    one instruction stream computes both: the rotations differ by a shift
//    register, Maj(a, b, c) = Ch(a ^ b, c, b) differs from Ch(e, f, g) =
//    Ch(~e, g, f) by one masked operation, and -d = (d ^ ~0) + 1 takes the
//    place of h + K + W (the a lanes read ones as their words).  The a lanes
//    run two steps behind: then both lanes want the partner's x1, a value one
//    step old, and the exchange (a DPP operand of the addition) waits for
//    nothing.  A step is 9 instructions -- 3 alignbit, 3 bitop3, xad, add, add3
//    -- against 14 for a round on one lane; the two steps of lag and the
//    selects at a block's ends add 26 to its 576.
//
// One 64 KiB chunk takes 1.18 ms (1.15 us per block, 4.6 cycles per
// instruction) against 1.79 with one lane per chunk and 2.65 with the one-wave
// kernel, whatever the number of chunks up to 64 per CU; up to 128 per CU 1.60
// against 1.88 and 2.69.
//
// A workgroup holds kGroups groups of 64 chunks, four waves each: two
// consumers of 32 chunks and two producers, which build alternate blocks and
// so have two block times for one block (a producer's 64 words are as many
// instructions as a consumer's block).  Up to 64 chunks per CU, one group per
// workgroup gives every wave a SIMD of its own.  Up to 128, two groups put one
// consumer and one producer on each SIMD (waves go to SIMDs in turn): 950
// instructions per SIMD and block, where two workgroups of one group could
// place two consumers on one.
//
// Synchronisation: every wave of the workgroup computes the same block count
// (the workgroup's most) and passes barriers 0..blocks.  Block b is produced
// between barriers b - 1 and b + 1 into buffer b % 3 and read into registers
// by the consumers after barrier b + 1; a consumer passes barrier b + 2 only
// when those reads have landed, and buffer b % 3 is next written after barrier
// b + 2.
//
// Exec mask: on gfx950 a wave whose rounds run with most lanes masked off is
// much slower per instruction than a full one (measured: 16 or fewer active
// lanes take about 1.6x as long per block as 32 or 64).  So every lane runs
// every block's expansion and rounds, also dead lanes and lanes past their
// last block (on zeros or stale words); only the loads, the state update and
// the digest store are per lane.
#include "hv_kernels.h"
#include "sha256_device.h"
#include "split_common.h"

#include <atomic>

namespace hv {
namespace {

constexpr uint32_t kRow = 65;  // a schedule row: 64 chunks' words, and the ones the a lanes add
constexpr int kMaxDevices = 64;

// The aligned dwords under block b of a chunk at p with nfull whole blocks and
// r tail bytes: only those holding at least one byte of the chunk are loaded
// (the others are zero), so no access leaves the pages the chunk touches.
// sh = p & 3, the same for every block of the chunk.
__device__ __forceinline__ uint32_t block_valid(uint32_t nfull, uint32_t r, uint32_t b) {
    return b < nfull ? 64u : (b == nfull ? r : 0u);
}

// The same from the chunk's byte count alone: 0 past its last byte.
__device__ __forceinline__ uint32_t valid_of(uint64_t nbytes, uint32_t b) {
    return block_valid((uint32_t)(nbytes >> 6), (uint32_t)(nbytes & 63), b);
}

// Block b's bytes into D.  kAligned (the chunk starts on a 16-byte boundary):
// the 16-byte granules that hold chunk bytes, with four 16-byte loads, into
// D[0..15] (D[16] is left as it is: with sh = 0 it does not enter the words).
// Otherwise the aligned dwords that hold chunk bytes, into D[0..16].  The
// others are zero.  An aligned granule or dword holding a chunk byte lies in
// the same page as that byte, so no access leaves the pages the chunk touches.
template <bool kAligned>
__device__ __forceinline__ void load_block(uint64_t src, uint32_t valid, uint32_t b, uint32_t D[17]) {
    if constexpr (kAligned) {
        const gquads q = reinterpret_cast<gquads>(src + 64 * (uint64_t)b);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if ((uint32_t)(16 * g) < valid) v = q[g];
            D[4 * g] = v.x; D[4 * g + 1] = v.y; D[4 * g + 2] = v.z; D[4 * g + 3] = v.w;
        }
    } else {
        const uint32_t sh = (uint32_t)(src & 3);
        const gwords w = reinterpret_cast<gwords>(src + 64 * (uint64_t)b - sh);
        const uint32_t end = valid > 0 ? sh + valid : 0u;  // no bytes: no loads, whatever the address
#pragma unroll
        for (int k = 0; k < 17; ++k) D[k] = (uint32_t)(4 * k) < end ? w[k] : 0u;
    }
}

// The 16 message words (big-endian) of block b from its dwords: a whole
// block, the tail block (tail, 0x80, zeros, and the bit length when r <= 55),
// or the length-only block that follows a tail of more than 55 bytes.
__device__ __forceinline__ void block_words(const uint32_t D[17], uint32_t sh, uint64_t total, uint32_t nfull,
                                            uint32_t r, uint32_t b, uint32_t W[16]) {
    const uint32_t valid = block_valid(nfull, r, b);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t x = __builtin_amdgcn_alignbyte(D[i + 1], D[i], sh);
        const int nv = (int)valid - 4 * i;  // bytes of the chunk in word i
        const uint32_t keep = nv >= 4 ? 0xffffffffu : (nv <= 0 ? 0u : (1u << (8 * nv)) - 1u);
        const uint32_t pad = (b == nfull && nv >= 0 && nv < 4) ? (0x80u << (8 * nv)) : 0u;
        W[i] = bswap((x & keep) | pad);
    }
    const bool last = b == nfull + (r <= 55 ? 0u : 1u);
    if (last) {
        const uint64_t bits = total * 8;
        W[14] = (uint32_t)(bits >> 32);
        W[15] = (uint32_t)bits;
    }
}

// The words of a whole block (no padding, no length).
__device__ __forceinline__ void whole_block_words(const uint32_t D[17], uint32_t sh, uint32_t W[16]) {
#pragma unroll
    for (int i = 0; i < 16; ++i) W[i] = bswap(__builtin_amdgcn_alignbyte(D[i + 1], D[i], sh));
}

// Producer p's blocks b = p, p + 2, ...: the loads of block b + 2 are issued,
// then block b's 64 schedule words, each with its round constant, go to buffer
// b % 3, half before barrier b and half before barrier b + 1.  Two register
// sets take turns, so that the loads run under the expansion and the barrier
// waits.  Every producer passes barriers 0..nmax.
template <bool kAligned>
__device__ __forceinline__ void produce_all(uint32_t p, uint64_t src, uint64_t total, uint32_t nfull, uint32_t r,
                                            uint32_t nblk, uint32_t nmax, uint32_t lane,
                                            uint4 (*sched)[16][kRow]) {
    const uint32_t sh = kAligned ? 0u : (uint32_t)(src & 3);
    uint32_t D[2][17];
#pragma unroll
    for (int k = 0; k < 17; ++k) D[0][k] = D[1][k] = 0;
    if (p < nblk) load_block<kAligned>(src, block_valid(nfull, r, p), p, D[0]);
    uint32_t passed = 0;  // barriers
    if (p == 1) {
        lds_barrier();
        ++passed;
    }
    uint32_t slot = p;  // b % 3
    for (uint32_t b0 = p; b0 < nmax; b0 += 4) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const uint32_t b = b0 + 2 * half;
            if (b < nmax) {
                uint32_t(&cur)[17] = D[half];
                uint32_t(&nxt)[17] = D[half ^ 1];
                wait_vmem();  // `cur` has landed; the loads below stay in flight
                if (b + 2 < nblk) load_block<kAligned>(src, block_valid(nfull, r, b + 2), b + 2, nxt);
                uint32_t W[16];
                if (__any(b - nfull < (r <= 55 ? 1u : 2u)))  // padding in this block of some chunk
                    block_words(cur, sh, total, nfull, r, b, W);
                else
                    whole_block_words(cur, sh, W);
                uint4(*buf)[kRow] = sched[slot];
                slot = slot == 0 ? 2 : slot - 1;  // (b + 2) % 3
#pragma unroll
                for (int g = 0; g < 16; ++g) {
                    uint32_t x[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int t = 4 * g + k;
                        if (t >= 16)
                            W[t & 15] = small_sigma1(W[(t - 2) & 15]) + W[(t - 7) & 15] +
                                        small_sigma0(W[(t - 15) & 15]) + W[t & 15];
                        x[k] = W[t & 15] + kRound[t];
                    }
                    buf[g][lane] = make_uint4(x[0], x[1], x[2], x[3]);
                    if (g == 8) lds_barrier();  // barrier b
                }
                lds_barrier();  // barrier b + 1: block b's words are in buf
                passed += 2;
            }
        }
    }
    for (; passed < nmax + 1; ++passed) lds_barrier();
}

// What tells the two lanes of a chunk apart.
struct Half {
    uint32_t r1, r2, r3;  // the lane's three rotations: Sigma0's (a lanes) or Sigma1's (e lanes)
    uint32_t m;           // ~0 in a lanes, 0 in e lanes
};

// Step s of the lanes' shared recurrence (see the top of the file): R[(i - s) & 3]
// is the lane's value i steps old, and the new value takes the oldest one's place.
// q: this step's -d or h + K + W and the partner's value, formed in the step
// before; its place is taken by the next step's (words next_kw).
//
// The order is fixed here: an instruction that needs the one before it issues
// 8 cycles after it, one that needs the second before 6 after that, and at a
// distance of four nothing is lost, so the nine are interleaved such that none
// needs the one before it.  The compiler's order had three that did, and waits
// before DPP operands: 1.31 us per block, 1.15 with this one and place_code.
#define HV_PIN __builtin_amdgcn_sched_barrier(0)
__device__ __forceinline__ uint32_t own_part(uint32_t x3, const Half& c, uint32_t kw) {
    uint32_t q;  // (x3 ^ m) + kw; the compiler would split this and share the addition with another
    asm("v_xad_u32 %0, %1, %2, %3" : "=v"(q) : "v"(x3), "v"(c.m), "v"(kw));
    return q;
}
// q plus the chunk's other lane's x1; written out for the same reason.  A DPP
// operand may be read no sooner than two instructions after it is written:
// `fresh` waits that out, elsewhere x1 is a step old.
template <bool fresh>
__device__ __forceinline__ uint32_t add_partner(uint32_t q, uint32_t x1) {
    uint32_t r;
    if constexpr (fresh)
        asm("s_nop 1\n\tv_add_u32_dpp %0, %1, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
            : "=v"(r) : "v"(x1), "v"(q));
    else
        asm("v_add_u32_dpp %0, %1, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(x1), "v"(q));
    return r;
}
__device__ __forceinline__ void step(uint32_t R[4], int s, const Half& c, uint32_t& q, uint32_t next_kw) {
    const uint32_t x0 = R[(0 - s) & 3], x1 = R[(1 - s) & 3], x2 = R[(2 - s) & 3];
    const uint32_t i = rotr(x0, c.r1);
    HV_PIN;
    const uint32_t j = rotr(x0, c.r2);
    HV_PIN;
    const uint32_t k = rotr(x0, c.r3);
    HV_PIN;
    const uint32_t p = __builtin_amdgcn_bitop3_b32(x0, x1, c.m, 0x2D);  // a ^ b, or ~e
    HV_PIN;
    const uint32_t sigma = xor3(i, j, k);
    HV_PIN;
    const uint32_t f = choose(p, x2, x1);  // Maj(a, b, c), or Ch(e, f, g)
    HV_PIN;
    const uint32_t next = own_part(x2, c, next_kw);
    HV_PIN;
    R[(3 - s) & 3] = sigma + f + q;
    HV_PIN;
    q = add_partner<false>(next, x0);
    HV_PIN;
}

// The place of the code that follows, all of it 8-byte instructions: on an
// 8-byte boundary a wave alone on its SIMD issues one every 4.6 cycles, and off
// it every 5.5 (1.18 ms for 64 KiB chunks, and 1.42).  Where a producer shares
// the SIMD it is off the boundary on purpose: the consumer, the older wave, is
// issued first, and at the full rate leaves its producer too few slots (1.89
// ms, and 1.59; with priority for the producer 1.78).
template <bool kAlone>
__device__ __forceinline__ void place_code() {
    HV_PIN;
    if constexpr (kAlone)
        asm volatile(".p2align 3");
    else
        asm volatile(".p2align 3\n\ts_nop 0");
    HV_PIN;
}

// The 64 rounds of one block on its words q (FIPS 180-4 section 6.2.2 steps
// 2-4): 64 steps of the e lanes, with the a lanes two steps behind.  H holds
// (H4, H5, H6, H7) in e lanes and (H2, H3, H0, H1) in a lanes, so that the
// values of step 64 feed forward into H[0] and H[1] in both; the feed-forward
// only where `on` (the lane still has blocks).
template <bool kAlone>
__device__ __forceinline__ void rounds(uint32_t H[4], const uint4 q[16], const Half& c, bool on) {
    uint32_t R[4] = {H[0], H[1], H[2], H[3]}, at64[4];
    uint32_t own = add_partner<true>(own_part(R[3], c, q[0].x), R[1]);
    place_code<kAlone>();
#pragma unroll
    for (int s = 0; s < 66; ++s) {
        const uint4 w = q[((s + 1) >> 2) & 15];
        const int k = (s + 1) & 3;
        const uint32_t next_kw = s + 1 >= 64 ? 1u : k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
        if (s == 64)
#pragma unroll
            for (int i = 0; i < 4; ++i) at64[i] = R[i];
        step(R, s, c, own, next_kw);
        // the a lanes' first two values are the block's b and a themselves
        if (s == 0) R[3] = c.m ? H[3] : R[3];
        if (s == 1) {
            R[2] = c.m ? H[2] : R[2];
            place_code<kAlone>();
        }
    }
#undef HV_PIN
    if (on) {
        H[0] += at64[0];
        H[1] += at64[1];
        H[2] += c.m ? R[2] : at64[2];
        H[3] += c.m ? R[3] : at64[3];
    }
}

// A consumer's work for block b (its words in `cur`): pass the barrier of
// block b + 1 and issue the reads of its words into `nxt`, then run block b's
// rounds, so the reads land under the rounds.  buf: b % 3, moved on.
template <bool kAlone>
__device__ __forceinline__ void consume(uint32_t b, uint32_t& buf, uint32_t nmax, uint32_t nblk, uint32_t col,
                                        uint4 (*sched)[16][kRow], uint32_t H[4], const Half& c, const uint4 cur[16],
                                        uint4 nxt[16]) {
    // `cur` has landed (read one block ago); waiting here, on every path and
    // before the next reads, keeps the compiler from placing a wait for it
    // where it would also wait for the reads issued below
    wait_lds();
    buf = buf == 2 ? 0 : buf + 1;
    if (b + 1 < nmax) {
        lds_barrier();  // barrier b + 2: block b + 1's words are in its buffer
#pragma unroll
        for (int g = 0; g < 16; ++g) nxt[g] = sched[buf][g][col];
    }
    rounds<kAlone>(H, cur, c, b < nblk);
}

template <int kGroups>
__global__ void __launch_bounds__(256 * kGroups) sha256_chain_kernel(const LeafDesc* __restrict__ desc,
                                                                     uint64_t n_slots, uint64_t out_bound,
                                                                     uint8_t* __restrict__ digests) {
    __shared__ uint4 sched[kGroups][3][16][kRow];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t group = (wave >> 1) % kGroups;
    const uint64_t base = ((uint64_t)blockIdx.x * kGroups + group) * 64;
    // every wave holds its group's 64 descriptors once, for the block counts
    uint64_t slot = base + lane;
    bool live = slot < n_slots;
    LeafDesc d = {0, 0, 0};
    if (live) d = desc[slot];
    uint32_t nfull = (uint32_t)(d.nbytes >> 6), r = (uint32_t)(d.nbytes & 63);
    uint32_t nblk = live ? nfull + (r <= 55 ? 1u : 2u) : 0u;
    // every wave of the workgroup runs the same number of barriers: the most
    // blocks of any of its chunks
    uint32_t nmax = nblk;
    if constexpr (kGroups == 2) {
        const uint64_t other = ((uint64_t)blockIdx.x * kGroups + (group ^ 1)) * 64 + lane;
        if (other < n_slots) {
            const uint64_t ob = desc[other].nbytes;
            const uint32_t on = (uint32_t)(ob >> 6) + ((ob & 63) <= 55 ? 1u : 2u);
            nmax = on > nmax ? on : nmax;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t x = __shfl_xor(nmax, o);
        nmax = x > nmax ? x : nmax;
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);

    if (wave >= 2 * kGroups) {
        // the ones of this producer's group (each writes half, before barrier 1)
        const uint32_t p = wave & 1;
        if (lane < 24) sched[group][(24 * p + lane) >> 4][(24 * p + lane) & 15][64] = make_uint4(1, 1, 1, 1);
        if (__all((d.src & 15) == 0))
            produce_all<true>(p, d.src, d.nbytes, nfull, r, nblk, nmax, lane, sched[group]);
        else
            produce_all<false>(p, d.src, d.nbytes, nfull, r, nblk, nmax, lane, sched[group]);
        return;
    }
    const uint32_t chunk = 32 * (wave & 1) + (lane >> 1);
    slot = base + chunk;
    live = slot < n_slots;
    if (live) d = desc[slot];
    nfull = (uint32_t)(d.nbytes >> 6);
    r = (uint32_t)(d.nbytes & 63);
    nblk = live ? nfull + (r <= 55 ? 1u : 2u) : 0u;
    const bool e = lane & 1;
    const Half c = {e ? 6u : 2u, e ? 11u : 13u, e ? 25u : 22u, e ? 0u : ~0u};
    uint32_t H[4] = {e ? kInit[4] : kInit[2], e ? kInit[5] : kInit[3], e ? kInit[6] : kInit[0],
                     e ? kInit[7] : kInit[1]};
    const uint32_t col = e ? chunk : 64u;
    // two register sets take turns: block b + 1's words are read into one
    // while block b's rounds run on the other
    uint4 A[16], B[16];
    if (nmax > 0) {
        lds_barrier();
        lds_barrier();  // block 0's words are in buffer 0
#pragma unroll
        for (int g = 0; g < 16; ++g) A[g] = sched[group][0][g][col];
    }
    uint32_t buf = 0;  // b % 3
    for (uint32_t b = 0; b < nmax; b += 2) {
        consume<kGroups == 1>(b, buf, nmax, nblk, col, sched[group], H, c, A, B);
        if (b + 1 < nmax) consume<kGroups == 1>(b + 1, buf, nmax, nblk, col, sched[group], H, c, B, A);
    }
    if (live && d.out < out_bound) {
        uint4* out = reinterpret_cast<uint4*>(digests + 32 * d.out);
        if (e)
            out[1] = make_uint4(bswap(H[0]), bswap(H[1]), bswap(H[2]), bswap(H[3]));
        else
            out[0] = make_uint4(bswap(H[2]), bswap(H[3]), bswap(H[0]), bswap(H[1]));
    }
}

// ---------------------------------------------------------------------------
// Three groups of 64 chunks per CU, one lane per chunk, for calls between 128
// and 192 chunks per CU.  A block's rounds are 903 instructions on its
// consumer and its words about 530 on a producer, so three groups are 1080 per
// SIMD if they are spread evenly.  A SIMD each for the consumers (waves 0-2)
// leaves the fourth to two producers (waves 3 and 7), which make two of the
// three groups' blocks; the third's comes from a helper on the SIMD of its
// consumer (waves 4-6), every third block, over three block times.  The two
// producers run at 4.8 cycles per instruction and the other SIMDs at 4.1, so
// the consumers make the last four words themselves: 36,800 chunks of 64 KiB
// take 2.29 ms without that, 2.13 with four words and 2.16 with eight (their
// own values are at hand, and nothing is sent).  Of two waves on a SIMD the
// older is issued first, and the younger producer then runs the second half
// of its block alone, at a lone wave's rate: with priority for the first 12 of
// its 15 entries 2.07 ms.  The one-wave kernel, a wave alone on each SIMD with
// 1405 instructions per block, takes 2.72.
//
// Interval u ends with barrier u.  Block b of a group is complete at barrier b
// (a producer's in interval b, a helper's, b % 3 == g, in b - 2 to b), is read
// into registers in interval b + 1 and run after barrier b + 1.  So a
// producer's buffer is busy for two intervals and a helper's for four, and
// three per group are enough (triple_buffer).

constexpr int kTriple = 3;
constexpr int kSent = 15;  // entries of four words a producer makes
constexpr int kAhead = 12;  // of these the younger producer makes with priority

// The schedule buffer of group g's block b: with k the count of the group's
// helper blocks before, they take buffers k % 3; a block after such a one
// takes (k + 2) % 3 and the next k % 3, free again by then.
__device__ __forceinline__ uint32_t triple_buffer(uint32_t b, uint32_t g) {
    const uint32_t k = (b + 9 - g) / 3, r = b + 9 - g - 3 * k;
    return (r == 1 ? k + 2 : k) % 3;
}

struct TripleLds {
    uint4 sched[kTriple][3][kSent][64];
    uint64_t src[kTriple][64], nbytes[kTriple][64];
};

// A producer's blocks b = first, first + stride, ..., block b for group g,
// which moves on by `turn` groups from block to block.  `younger`: wave 7.
template <bool kAligned>
__device__ __forceinline__ void triple_produce(uint32_t first, uint32_t stride, uint32_t g, uint32_t turn,
                                               bool younger, uint32_t nmax, uint32_t lane, TripleLds& lds) {
    uint32_t D[2][17];
#pragma unroll
    for (int k = 0; k < 17; ++k) D[0][k] = D[1][k] = 0;
    uint64_t src = lds.src[g][lane], total = lds.nbytes[g][lane];
    if (first < nmax) load_block<kAligned>(src, valid_of(total, first), first, D[0]);
    uint32_t passed = 0;  // barriers
    for (uint32_t b0 = first; b0 < nmax; b0 += 2 * stride) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const uint32_t b = b0 + half * stride;
            if (b < nmax) {
                if (younger) __builtin_amdgcn_s_setprio(1);
                const uint32_t after = g + turn < kTriple ? g + turn : g + turn - kTriple;
                const uint64_t src1 = lds.src[after][lane], total1 = lds.nbytes[after][lane];
                uint32_t(&cur)[17] = D[half];
                wait_vmem();  // `cur` has landed; the loads below stay in flight
                load_block<kAligned>(src1, valid_of(total1, b + stride), b + stride, D[half ^ 1]);
                const uint32_t sh = kAligned ? 0u : (uint32_t)(src & 3);
                const uint32_t nfull = (uint32_t)(total >> 6), r = (uint32_t)(total & 63);
                uint32_t W[16];
                if (__any(b - nfull < (r <= 55 ? 1u : 2u)))  // padding in this block of some chunk
                    block_words(cur, sh, total, nfull, r, b, W);
                else
                    whole_block_words(cur, sh, W);
                uint4(*buf)[64] = lds.sched[g][triple_buffer(b, g)];
#pragma unroll
                for (int q = 0; q < kSent; ++q) {
#pragma unroll
                    for (int t = 4 * q; t < 4 * q + 4; ++t)
                        if (t >= 16)
                            W[t & 15] = small_sigma1(W[(t - 2) & 15]) + W[(t - 7) & 15] +
                                        small_sigma0(W[(t - 15) & 15]) + W[t & 15];
                    buf[q][lane] = make_uint4(W[(4 * q) & 15], W[(4 * q + 1) & 15], W[(4 * q + 2) & 15],
                                              W[(4 * q + 3) & 15]);
                    if (younger && q == kAhead - 1) __builtin_amdgcn_s_setprio(0);
                    // a helper's thirds of a block
                    if ((q == 6 && passed + 1 < b) || (q == 10 && passed < b)) {
                        lds_barrier();
                        ++passed;
                    }
                }
                lds_barrier();  // barrier b
                ++passed;
                src = src1;
                total = total1;
                g = after;
            }
        }
    }
    for (; passed < nmax; ++passed) lds_barrier();
}

__device__ __forceinline__ void triple_consume(uint32_t b, uint32_t g, uint32_t nmax, uint32_t nblk, uint32_t lane,
                                               TripleLds& lds, uint32_t H[8], const uint4 cur[kSent], uint4 nxt[kSent]) {
    wait_lds();  // `cur` has landed; here, so that no wait for it also waits for the reads below
    if (b + 1 < nmax) {
        lds_barrier();  // barrier b + 1
        uint4(*buf)[64] = lds.sched[g][triple_buffer(b + 1, g)];
#pragma unroll
        for (int q = 0; q < kSent; ++q) nxt[q] = buf[q][lane];
    }
    uint32_t s[8], W[64];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = H[i];
#pragma unroll
    for (int q = 0; q < kSent; ++q) {
        W[4 * q] = cur[q].x; W[4 * q + 1] = cur[q].y; W[4 * q + 2] = cur[q].z; W[4 * q + 3] = cur[q].w;
    }
#pragma unroll
    for (int t = 0; t < 64; ++t) {
        if (t >= 4 * kSent) W[t] = small_sigma1(W[t - 2]) + W[t - 7] + small_sigma0(W[t - 15]) + W[t - 16];
        const uint32_t w = W[t];
        const uint32_t e = s[(12 - t) & 7], a = s[(8 - t) & 7];
        const uint32_t t1 = s[(15 - t) & 7] + kRound[t] + w + big_sigma1(e) +
                            choose(e, s[(13 - t) & 7], s[(14 - t) & 7]);
        const uint32_t t2 = big_sigma0(a) + majority(a, s[(9 - t) & 7], s[(10 - t) & 7]);
        s[(11 - t) & 7] += t1;
        s[(15 - t) & 7] = t1 + t2;
    }
    // a select: under a branch the compiler would move the rounds there too
    const uint32_t on = b < nblk ? ~0u : 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) H[i] += s[i] & on;
}

__global__ void __launch_bounds__(512) sha256_triple_kernel(const LeafDesc* __restrict__ desc, uint64_t n_slots,
                                                            uint64_t out_bound, uint8_t* __restrict__ digests) {
    __shared__ TripleLds lds;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t base = (uint64_t)blockIdx.x * (64 * kTriple);
    // every wave counts the workgroup's blocks
    uint32_t nmax = 0;
    bool aligned = true;
#pragma unroll
    for (int g = 0; g < kTriple; ++g) {
        const uint64_t slot = base + 64 * g + lane;
        LeafDesc d = {0, 0, 0};
        if (slot < n_slots) {
            d = desc[slot];
            const uint32_t nfull = (uint32_t)(d.nbytes >> 6);
            const uint32_t nblk = nfull + ((d.nbytes & 63) <= 55 ? 1u : 2u);
            nmax = nblk > nmax ? nblk : nmax;
            aligned = aligned && (d.src & 15) == 0;
        }
        if (wave == g) {
            lds.src[g][lane] = d.src;
            lds.nbytes[g][lane] = d.nbytes;
        }
    }
    aligned = __all(aligned);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t x = __shfl_xor(nmax, o);
        nmax = x > nmax ? x : nmax;
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);
    lds_barrier();  // the descriptors are in LDS

    if (wave >= kTriple) {
        const bool helper = wave != 3 && wave != 7;
        // block 0: waves 3 and 7 make groups 1 and 2, the helper of group 0 the other
        const uint32_t g = wave == 3 ? 1u : wave == 7 ? 2u : wave - 4;
        const uint32_t first = helper ? g : 0u, stride = helper ? 3u : 1u, turn = helper ? 0u : 1u;
        if (aligned)
            triple_produce<true>(first, stride, g, turn, wave == 7, nmax, lane, lds);
        else
            triple_produce<false>(first, stride, g, turn, wave == 7, nmax, lane, lds);
        return;
    }
    const uint64_t slot = base + 64 * wave + lane;
    const bool live = slot < n_slots;
    const uint64_t total = lds.nbytes[wave][lane];
    const uint32_t nblk = live ? (uint32_t)(total >> 6) + ((total & 63) <= 55 ? 1u : 2u) : 0u;
    __builtin_amdgcn_s_setprio(2);  // over the helper's, whose thirds are due no sooner
    uint32_t H[8];
    init_state(H);
    uint4 A[kSent], B[kSent];
    if (nmax > 0) {
        lds_barrier();  // barrier 0
        uint4(*buf)[64] = lds.sched[wave][triple_buffer(0, wave)];
#pragma unroll
        for (int q = 0; q < kSent; ++q) A[q] = buf[q][lane];
    }
    for (uint32_t b = 0; b < nmax; b += 2) {
        triple_consume(b, wave, nmax, nblk, lane, lds, H, A, B);
        if (b + 1 < nmax) triple_consume(b + 1, wave, nmax, nblk, lane, lds, H, B, A);
    }
    if (live) {
        const uint64_t out = desc[slot].out;
        if (out < out_bound) store_digest(digests + 32 * out, H);
    }
}

}  // namespace

// Compute units of the current device, queried once per device.
uint32_t device_cus() {
    static std::atomic<int> cus[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    int n = cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 0;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return (uint32_t)n;
}

int leaf_launch_for(int alg, uint64_t n_slots, bool background, uint64_t cus) {
    const int choice = leaf_kernel_choice();
    // the chain kernels while every CU holds one workgroup at most: 64
    // KiB chunks take 1.18 ms up to 64 per CU and 1.60 up to 128, against 2.69
    // with the one-wave kernel; with more, two workgroups share a CU and the
    // one-wave kernel (or SHA-256's three-group one) is
    // faster.  Background work keeps the one-wave kernel: beside decode-shaped
    // products a chain kernel scans 2.2 times as fast and costs them 1.8 times
    // as much at slices of 4,096 chunks (15.4% against 8.5%), 7 times at 16,384
    // (80% against 11%).
    if (choice == 1 || (choice == 0 && (background || n_slots > 128 * cus))) {
        // SHA-256, up to three groups per CU, one workgroup each: 2.07 ms
        // against 2.72 for 64 KiB chunks (above kSent); with more, the one-wave
        // kernel has a wave for every SIMD
        const bool three = alg == kAlgSha256 && choice == 0 && !background && n_slots <= 64 * kTriple * cus;
        return three ? kLeafThreeGroup : kLeafOneWave;
    }
    return choice == 3 || n_slots > 64 * cus ? kLeafTwoWaveCompact : kLeafTwoWave;
}

uint32_t tape_waves(uint64_t n_slots, uint32_t cus) {
    // In units of a wave's time when a SIMD is full: one wave alone on a SIMD
    // takes 1.10 (64 KiB chunks: 2.72 ms), two 2.04 (5.06), three 3 (7.44), and
    // a fourth waits for one of them (SHA-384: 3.51, 6.35 and 9.30 ms, 1.13, 2.05
    // and 3; nearly the same choices).  x waves per SIMD run plainly as threes
    // and a remainder; on a tape, as w at once (at most x: an interval is no
    // shorter than a chunk), each x / w long.
    static constexpr double kAtOnce[4] = {0, 1.10, 2.04, 3.0};
    const uint32_t simds = 4 * cus;
    if (simds == 0 || 3 * simds > kTapeMaxWaves) return 0;
    const double x = (double)n_slots / 64 / simds;
    const uint64_t whole = (n_slots + 64 * (uint64_t)simds - 1) / (64 * (uint64_t)simds);
    double best = ((double)(whole / 3 * 3) + kAtOnce[whole % 3]) * 0.96;  // the walk's own cost
    uint32_t waves = 0;
    for (uint32_t w = 1; w <= 3 && w <= x; ++w)
        if (x / w * kAtOnce[w] < best) {
            best = x / w * kAtOnce[w];
            waves = w * simds;
        }
    return waves;
}

hipError_t launch_sha256_auto(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              hipStream_t s, bool background) {
    const int k = leaf_launch_for(kAlgSha256, n_slots, background, device_cus());
    if (k == kLeafThreeGroup) {
        sha256_triple_kernel<<<(unsigned)((n_slots + 64 * kTriple - 1) / (64 * kTriple)), 512, 0, s>>>(
            desc, n_slots, out_bound, digests);
        return hipGetLastError();
    }
    if (k == kLeafOneWave) return launch_sha256_leaves(desc, n_slots, out_bound, digests, s);
    return launch_sha256_split(desc, n_slots, out_bound, digests, k == kLeafTwoWaveCompact, s);
}

hipError_t launch_sha256_split(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                               bool two_groups, hipStream_t s) {
    for (uint64_t base = 0; base < n_slots; base += kMaxSlotsPerLaunch) {
        const uint64_t n = n_slots - base < kMaxSlotsPerLaunch ? n_slots - base : kMaxSlotsPerLaunch;
        if (!two_groups)
            sha256_chain_kernel<1><<<(unsigned)((n + 63) / 64), 256, 0, s>>>(desc + base, n, out_bound, digests);
        else
            sha256_chain_kernel<2><<<(unsigned)((n + 127) / 128), 512, 0, s>>>(desc + base, n, out_bound, digests);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace hv
