// sha384_split.hip -- SHA-384 of every chunk for small leaf counts: the
// SHA-384 forms of the kernels that shorten one chunk's chain of blocks
// (sha256_split.hip).
//
// A chunk is one chain of 128-byte blocks, so with fewer chunks than the chip
// has lanes its time is that chain's latency, and a lone wave issues one
// instruction per 4.6 to 4.9 cycles: the instructions on the wave that carries
// the state are the time.  The one-wave kernel has 3416 per block.
//
// Up to 64 chunks per CU: the chain kernel.  A chunk has two lanes of a
// consumer wave, one for a..d and one for e..h, whose halves of a round are
// one instruction stream with the a lanes two steps behind (the recurrence is
// explained in sha256_split.hip), and two producer waves build alternate
// blocks' 80 schedule words, each with its round constant.  On 64-bit words
// in 32-bit halves a step is 19 instructions against 27 for a round on one
// lane: a Sigma 8 (as rotr(x ^ rotr(x, i) ^ rotr(x, j), k), whose amounts are
// below 32 for Sigma0 and Sigma1 alike, so that the two lanes' rotations
// differ by a shift register only), Ch or Maj 4, -d or h + K + W 3, the
// partner's value 2 (an addition with DPP operands) and 2 additions.  A
// workgroup is 64 chunks, two consumers and two producers, a SIMD each; three
// buffers of 40 x 65 16-byte entries are 122 KB of its CU's LDS.
// 9,225 chunks of 256 KiB, with the reductions above them: 6.24 ms (3.0 us and
// 1570 instructions per block) against 9.39 with one lane per chunk and one
// producer (2163 instructions).  The compiler's order of a step took 6.66.
//
// Up to 128 chunks per CU: the two-pair kernel, one lane per chunk.  A
// producer wave loads each block one block ahead, builds its 16 message words
// (padding of FIPS 180-4 section 5.1.2: tail, 0x80, zeros, 128-bit bit length)
// and expands them to the 80 schedule words (section 6.4 step 1) in a
// double-buffered LDS area; a consumer wave runs only the 80 rounds and the
// feed-forward.  Two pairs' schedules, 80 x 8 bytes per lane and buffer, fill
// the CU's 160 KB of LDS.
//
// Synchronisation and exec mask: the chain kernel's barriers are those of the
// SHA-256 one; both waves of a pair of the two-pair kernel run one barrier per
// block (the workgroup's most blocks).  Barriers order LDS only.  Every lane
// runs every block (dead lanes and finished chunks on zeros or stale words)
// and only the loads, the state update and the digest store are per lane.
#include "hv_kernels.h"
#include "sha384_device.h"
#include "split_common.h"

namespace hv {
namespace {

constexpr int kEntries = 40;  // 80 schedule words, two per 16-byte LDS entry
constexpr int kRow = 65;       // a schedule row of the chain kernel: 64 chunks' entries, and the ones the a lanes add

__device__ __forceinline__ uint32_t block_valid(uint32_t nfull, uint32_t r, uint32_t b) {
    return b < nfull ? 128u : (b == nfull ? r : 0u);
}

// Block b's bytes into D, as in the SHA-256 kernel: kAligned (16-byte aligned
// chunk) loads the 16-byte granules holding chunk bytes into D[0..31] (D[32]
// is left as it is: with sh = 0 it does not enter the words), otherwise the
// aligned dwords holding chunk bytes into D[0..32]; the others are zero.  An
// aligned granule or dword holding a chunk byte lies in that byte's page.
template <bool kAligned>
__device__ __forceinline__ void load_block(uint64_t src, uint32_t valid, uint32_t b, uint32_t D[33]) {
    if constexpr (kAligned) {
        const gquads q = reinterpret_cast<gquads>(src + 128 * (uint64_t)b);
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if ((uint32_t)(16 * g) < valid) v = q[g];
            D[4 * g] = v.x; D[4 * g + 1] = v.y; D[4 * g + 2] = v.z; D[4 * g + 3] = v.w;
        }
    } else {
        const uint32_t sh = (uint32_t)(src & 3);
        const gwords w = reinterpret_cast<gwords>(src + 128 * (uint64_t)b - sh);
        const uint32_t end = valid > 0 ? sh + valid : 0u;  // no bytes: no loads, whatever the address
#pragma unroll
        for (int k = 0; k < 33; ++k) D[k] = (uint32_t)(4 * k) < end ? w[k] : 0u;
    }
}

// The 16 message words of a whole block.
__device__ __forceinline__ void whole_block_words(const uint32_t D[33], uint32_t sh, uint64_t W[16]) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
        W[i] = be64(__builtin_amdgcn_alignbyte(D[2 * i + 1], D[2 * i], sh),
                    __builtin_amdgcn_alignbyte(D[2 * i + 2], D[2 * i + 1], sh));
}

// The 16 message words of block b of a chunk of `total` bytes with nfull
// whole blocks and r tail bytes: a whole block, the tail block (and the bit
// length when r <= 111), or the length-only block after a longer tail.
__device__ __forceinline__ void block_words(const uint32_t D[33], uint32_t sh, uint64_t total, uint32_t nfull,
                                            uint32_t r, uint32_t b, uint64_t W[16]) {
    const uint32_t valid = block_valid(nfull, r, b);
    uint32_t X[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const uint32_t x = __builtin_amdgcn_alignbyte(D[i + 1], D[i], sh);
        const int nv = (int)valid - 4 * i;  // bytes of the chunk in dword i
        const uint32_t keep = nv >= 4 ? 0xffffffffu : (nv <= 0 ? 0u : (1u << (8 * nv)) - 1u);
        const uint32_t pad = (b == nfull && nv >= 0 && nv < 4) ? (0x80u << (8 * nv)) : 0u;
        X[i] = (x & keep) | pad;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) W[i] = be64(X[2 * i], X[2 * i + 1]);
    if (b == nfull + (r <= 111 ? 0u : 1u)) {
        W[14] = total >> 61;
        W[15] = total << 3;
    }
}

// Two 64-bit words as one 16-byte LDS entry, and back.
__device__ __forceinline__ uint4 entry(uint64_t w0, uint64_t w1) {
    return make_uint4(lo32(w0), hi32(w0), lo32(w1), hi32(w1));
}

// Producer: issue block b + 1's loads into `nxt`, build block b's 80
// schedule words from `cur` into `buf` (16 message words, then four trips of
// 16 expanded words), meet the consumer at the barrier.
template <bool kAligned>
__device__ __forceinline__ void produce(uint32_t b, uint64_t src, uint64_t total, uint32_t nfull, uint32_t r,
                                        uint32_t nblk, uint32_t nfull_min, uint32_t lane, uint4 (*buf)[64],
                                        const uint32_t cur[33], uint32_t nxt[33]) {
    const uint32_t sh = kAligned ? 0u : (uint32_t)(src & 3);
    // `cur` has landed (its loads were issued one block ago); waiting here,
    // before the next loads, keeps the compiler from waiting for those too
    wait_vmem();
    if (b + 1 < nblk) load_block<kAligned>(src, block_valid(nfull, r, b + 1), b + 1, nxt);
    uint64_t W[16];
    if (b < nfull_min)  // wave-uniform: a whole block on every lane
        whole_block_words(cur, sh, W);
    else
        block_words(cur, sh, total, nfull, r, b, W);
#pragma unroll
    for (int g = 0; g < 8; ++g) buf[g][lane] = entry(W[2 * g], W[2 * g + 1]);
#pragma nounroll
    for (int trip = 1; trip < 5; ++trip) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            W[i] = small_sigma1_512(W[(i + 14) & 15]) + W[(i + 9) & 15] + small_sigma0_512(W[(i + 1) & 15]) + W[i];
#pragma unroll
        for (int g = 0; g < 8; ++g) buf[8 * trip + g][lane] = entry(W[2 * g], W[2 * g + 1]);
    }
    lds_barrier();  // block b's words are in buf
}

template <bool kAligned>
__device__ __forceinline__ void produce_all(uint64_t src, uint64_t total, uint32_t nfull, uint32_t r, uint32_t nblk,
                                            uint32_t nmax, uint32_t nfull_min, uint32_t lane,
                                            uint4 (*sched)[kEntries][64]) {
    uint32_t A[33], B[33];
#pragma unroll
    for (int k = 0; k < 33; ++k) A[k] = B[k] = 0;
    if (0 < nblk) load_block<kAligned>(src, block_valid(nfull, r, 0), 0, A);
    for (uint32_t b = 0; b < nmax; b += 2) {
        produce<kAligned>(b, src, total, nfull, r, nblk, nfull_min, lane, sched[0], A, B);
        if (b + 1 < nmax) produce<kAligned>(b + 1, src, total, nfull, r, nblk, nfull_min, lane, sched[1], B, A);
    }
}

__global__ void __launch_bounds__(256) sha384_pairs_kernel(const LeafDesc* __restrict__ desc, uint64_t n_slots,
                                                           uint64_t out_bound, uint8_t* __restrict__ digests) {
    // [pair][buffer][entry of two words][lane]
    __shared__ uint4 sched[2][2][kEntries][64];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t pair = wave >> 1;
    const uint64_t base = (uint64_t)blockIdx.x * 128;
    const uint64_t slot = base + 64 * pair + lane;
    const bool live = slot < n_slots;
    LeafDesc d = {0, 0, 0};
    if (live) d = desc[slot];
    const uint32_t nfull = (uint32_t)(d.nbytes >> 7);
    const uint32_t r = (uint32_t)(d.nbytes & 127);
    const uint32_t nblk = live ? nfull + (r <= 111 ? 1u : 2u) : 0u;
    // every wave of the workgroup runs the same number of barriers: the most
    // blocks of any of its chunks
    uint32_t nmax = nblk;
    const uint64_t other = base + 64 * (pair ^ 1) + lane;
    if (other < n_slots) {
        const uint64_t ob = desc[other].nbytes;
        const uint32_t on = (uint32_t)(ob >> 7) + ((ob & 127) <= 111 ? 1u : 2u);
        nmax = on > nmax ? on : nmax;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t x = __shfl_xor(nmax, o);
        nmax = x > nmax ? x : nmax;
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);

    if ((wave & 1) == 0) {
        uint32_t nfull_min = live ? nfull : 0xffffffffu;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const uint32_t x = __shfl_xor(nfull_min, o);
            nfull_min = x < nfull_min ? x : nfull_min;
        }
        nfull_min = __builtin_amdgcn_readfirstlane(nfull_min);
        if (__all((d.src & 15) == 0))
            produce_all<true>(d.src, d.nbytes, nfull, r, nblk, nmax, nfull_min, lane, sched[pair]);
        else
            produce_all<false>(d.src, d.nbytes, nfull, r, nblk, nmax, nfull_min, lane, sched[pair]);
    } else {
        uint64_t H[8];
        init_state384(H);
        for (uint32_t b = 0; b < nmax; ++b) {
            lds_barrier();  // block b's words are in buffer b % 2
            uint4(*buf)[64] = sched[pair][b & 1];
            uint64_t s[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) s[i] = H[i];
            // the words in five groups of 16 (eight entries): group j + 1's
            // reads are issued before group j's rounds; the scheduling barrier
            // keeps the compiler from moving each read next to its use, where
            // its latency would stall the rounds
            uint4 q[2][8];
#pragma unroll
            for (int e = 0; e < 8; ++e) q[0][e] = buf[e][lane];
#pragma unroll
            for (int j = 0; j < kEntries / 8; ++j) {
                if (j + 1 < kEntries / 8) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) q[(j + 1) & 1][e] = buf[8 * (j + 1) + e][lane];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint64_t w2[2] = {pack(q[j & 1][e].y, q[j & 1][e].x), pack(q[j & 1][e].w, q[j & 1][e].z)};
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int t = 16 * j + 2 * e + k;
                        round512(s[(8 - t) & 7], s[(9 - t) & 7], s[(10 - t) & 7], s[(11 - t) & 7],
                                 s[(12 - t) & 7], s[(13 - t) & 7], s[(14 - t) & 7], s[(15 - t) & 7], kRound512[t],
                                 w2[k]);
                    }
                }
            }
            const bool on = b < nblk;
#pragma unroll
            for (int i = 0; i < 8; ++i) H[i] = on ? H[i] + s[i] : H[i];
        }
        if (live && d.out < out_bound) store_digest384(digests + 48 * d.out, H);
    }
}

// Producer p's blocks b = p, p + 2, ... of the chain kernel: as produce_all,
// but each word with its round constant, into buffer b % 3, three fifths of a
// block before barrier b and the rest before barrier b + 1.  Every producer
// passes barriers 0..nmax.
template <bool kAligned>
__device__ __forceinline__ void produce_alternate(uint32_t p, uint64_t src, uint64_t total, uint32_t nfull, uint32_t r,
                                                  uint32_t nblk, uint32_t nmax, uint32_t lane,
                                                  uint4 (*sched)[kEntries][kRow]) {
    const uint32_t sh = kAligned ? 0u : (uint32_t)(src & 3);
    uint32_t D[2][33];
#pragma unroll
    for (int k = 0; k < 33; ++k) D[0][k] = D[1][k] = 0;
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
                uint32_t(&cur)[33] = D[half];
                uint32_t(&nxt)[33] = D[half ^ 1];
                wait_vmem();  // `cur` has landed; the loads below stay in flight
                if (b + 2 < nblk) load_block<kAligned>(src, block_valid(nfull, r, b + 2), b + 2, nxt);
                uint64_t W[16];
                if (__any(b - nfull < (r <= 111 ? 1u : 2u)))  // padding in this block of some chunk
                    block_words(cur, sh, total, nfull, r, b, W);
                else
                    whole_block_words(cur, sh, W);
                uint4(*buf)[kRow] = sched[slot];
                slot = slot == 0 ? 2 : slot - 1;  // (b + 2) % 3
#pragma unroll
                for (int g = 0; g < 8; ++g)
                    buf[g][lane] = entry(W[2 * g] + kRound512[2 * g], W[2 * g + 1] + kRound512[2 * g + 1]);
#pragma nounroll
                for (int trip = 1; trip < 5; ++trip) {
                    if (trip == 3) lds_barrier();  // barrier b
                    const uint64_t* k = kRound512 + 16 * trip;
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        W[i] = small_sigma1_512(W[(i + 14) & 15]) + W[(i + 9) & 15] +
                               small_sigma0_512(W[(i + 1) & 15]) + W[i];
#pragma unroll
                    for (int g = 0; g < 8; ++g)
                        buf[8 * trip + g][lane] = entry(W[2 * g] + k[2 * g], W[2 * g + 1] + k[2 * g + 1]);
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
    uint32_t r1, r2, r3;  // the lane's rotations: rotr(x ^ rotr(x, r1) ^ rotr(x, r2), r3) is its Sigma
    uint32_t m;           // ~0 in a lanes, 0 in e lanes
};

__device__ __forceinline__ uint64_t rotr64_below_32(uint64_t x, uint32_t n) {
    return pack(__builtin_amdgcn_alignbit(lo32(x), hi32(x), n), __builtin_amdgcn_alignbit(hi32(x), lo32(x), n));
}

#define HV_PIN __builtin_amdgcn_sched_barrier(0)

// (x3 ^ m) + kw: a step's -d, or h + K + W.
__device__ __forceinline__ uint64_t own_part(uint64_t x3, const Half& c, uint64_t kw) {
    // the XOR as an 8-byte instruction (see place_code)
    const uint64_t x = pack(__builtin_amdgcn_bitop3_b32(hi32(x3), c.m, c.m, 0x3C),
                            __builtin_amdgcn_bitop3_b32(lo32(x3), c.m, c.m, 0x3C));
    HV_PIN;
    return x + kw;
}

// x plus the chunk's other lane's y, in two halves: the low words' sum leaves
// its carry in VCC, and the high words' sum takes it from there.  Two things
// the hardware does not wait for and the compiler, which does not see into the
// blocks, does not add waits for: VCC may be read by a vector instruction no
// sooner than two instructions after one wrote it, so the halves have at least
// two instructions between them (the blocks are volatile, which keeps their
// order with others), and a DPP operand no sooner than two after it is written
// (`fresh` waits that out, elsewhere y is a step old).
// tests/test_isa_waits.py reads both distances in the kernel's code.
__device__ __forceinline__ uint32_t add_partner_low(uint32_t x, uint32_t y, uint64_t& carry) {
    uint32_t r;
    register uint64_t vcc asm("vcc");
    asm volatile("v_add_co_u32_dpp %0, vcc, %2, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
                 : "=v"(r), "=s"(vcc) : "v"(y), "v"(x));
    carry = vcc;
    return r;
}
__device__ __forceinline__ uint32_t add_partner_high(uint32_t x, uint32_t y, uint64_t carry) {
    uint32_t r;
    register uint64_t vcc asm("vcc") = carry;  // written too
    asm volatile("v_addc_co_u32_dpp %0, vcc, %2, %3, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
                 : "=v"(r), "+s"(vcc) : "v"(y), "v"(x));
    return r;
}
// Both at once, with the waits.
__device__ __forceinline__ uint64_t add_partner_fresh(uint64_t x, uint64_t y) {
    uint32_t lo, hi;
    asm("s_nop 1\n\tv_add_co_u32_dpp %0, vcc, %2, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_addc_co_u32_dpp %1, vcc, %4, %5, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
        : "=&v"(lo), "=v"(hi) : "v"(lo32(y)), "v"(lo32(x)), "v"(hi32(y)), "v"(hi32(x)) : "vcc");
    return pack(hi, lo);
}

// Step s of the lanes' shared recurrence: R[(i - s) & 3] is the lane's value i
// steps old, and the new value takes the oldest one's place.  q: this step's
// -d or h + K + W and the partner's value, formed in the step before; its place
// is taken by the next step's (word next_kw).  The order is fixed, as in
// sha256_split.hip, with two or more instructions between any and the one that
// needs it, except the last addition's t.  (With the halves of the partner's
// addition next to each other and t before them, the same time: 9,225 chunks of
// 256 KiB 5.96 ms, 5.95 in this order.)
template <int s>
__device__ __forceinline__ void step(uint64_t R[4], const Half& c, uint64_t& q, uint64_t next_kw) {
    const uint64_t x0 = R[(0 - s) & 3], x1 = R[(1 - s) & 3], x2 = R[(2 - s) & 3];
    const uint64_t n = pack(__builtin_amdgcn_bitop3_b32(hi32(x2), c.m, c.m, 0x3C),
                            __builtin_amdgcn_bitop3_b32(lo32(x2), c.m, c.m, 0x3C));  // as own_part
    HV_PIN;
    const uint64_t i = rotr64_below_32(x0, c.r1);
    HV_PIN;
    const uint64_t j = rotr64_below_32(x0, c.r2);
    HV_PIN;
    const uint64_t own = n + next_kw;
    HV_PIN;
    const uint64_t p = bitop3_64<0x2D>(x0, x1, pack(c.m, c.m));  // a ^ b, or ~e
    HV_PIN;
    const uint64_t y = bitop3_64<0x96>(x0, i, j);
    HV_PIN;
    uint64_t carry = 0;
    uint32_t low = 0;
    if constexpr (s < 81) low = add_partner_low(lo32(own), lo32(x0), carry);
    HV_PIN;
    uint64_t f = bitop3_64<0xCA>(p, x2, x1);  // Maj(a, b, c), or Ch(e, f, g)
    // where a branch follows the step, the compiler would move this behind it,
    // and the halves would be neighbours.  (With waits there instead, which are 4
    // bytes each and shift what follows: 26 chunks of 128 KiB 2.94 ms, so 2.92.)
    if constexpr (s == 63 || s == 80) asm volatile("" : "+v"(f));
    HV_PIN;
    const uint64_t sigma = rotr64_below_32(y, c.r3);
    HV_PIN;
    const uint64_t t = f + q;
    HV_PIN;
    if constexpr (s < 81) q = pack(add_partner_high(hi32(own), hi32(x0), carry), low);
    HV_PIN;
    R[(3 - s) & 3] = sigma + t;
    HV_PIN;
}

// The place of the code that follows, all of it 8-byte instructions: on an
// 8-byte boundary a wave alone on its SIMD issues faster (sha256_split.hip).
__device__ __forceinline__ void place_code() {
    HV_PIN;
    asm volatile(".p2align 3");
    HV_PIN;
}

// Steps s to end - 1, word s + 1 of the schedule (a pair per entry) from `q`, or
// from `after` for the first of the next sixteen (ones after the last).
template <int s, int end>
__device__ __forceinline__ void steps(uint64_t R[4], const uint64_t H[4], const Half& c, uint64_t& own,
                                      const uint4 q[8], const uint4 after[8]) {
    if constexpr (s < end) {
        const uint4 w = s + 1 < end ? q[((s + 1) >> 1) & 7] : after[0];
        step<s>(R, c, own, s + 1 >= 80 ? 1 : s & 1 ? pack(w.y, w.x) : pack(w.w, w.z));
        // the a lanes' first two values are the block's b and a themselves
        if (s == 0) R[3] = c.m ? H[3] : R[3];
        if (s == 1) {
            R[2] = c.m ? H[2] : R[2];
            place_code();
        }
        steps<s + 1, end>(R, H, c, own, q, after);
    }
}

// A consumer's work for block b: 80 steps of the e lanes with the a lanes two
// steps behind, the words in five groups of 16.  `cur` is being read on entry;
// group j + 1's reads (after group 4 those of block b + 1, past its barrier)
// are issued before group j's steps, which the scheduling barrier keeps there,
// and land under them.  H holds (H4, H5, H6, H7) in e lanes and (H2, H3, H0,
// H1) in a lanes; slot: b % 3, moved on.
__device__ __forceinline__ void consume(uint32_t b, uint32_t& slot, uint32_t nmax, uint32_t nblk, uint32_t col,
                                        uint4 (*sched)[kEntries][kRow], uint64_t H[4], const Half& c, uint4 cur[8],
                                        uint4 nxt[8]) {
    uint64_t R[4] = {H[0], H[1], H[2], H[3]};
    auto read = [&](uint32_t from, int j, uint4 q[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = sched[from][8 * j + e][col];
    };
    wait_lds();
    uint64_t own = add_partner_fresh(own_part(R[3], c, pack(cur[0].y, cur[0].x)), R[1]);
    read(slot, 1, nxt);
    place_code();
    steps<0, 16>(R, H, c, own, cur, nxt);
    wait_lds();
    read(slot, 2, cur);
    place_code();
    steps<16, 32>(R, H, c, own, nxt, cur);
    wait_lds();
    read(slot, 3, nxt);
    place_code();
    steps<32, 48>(R, H, c, own, cur, nxt);
    wait_lds();
    read(slot, 4, cur);
    place_code();
    steps<48, 64>(R, H, c, own, nxt, cur);
    wait_lds();
    slot = slot == 2 ? 0 : slot + 1;
    if (b + 1 < nmax) {
        lds_barrier();  // barrier b + 2: block b + 1's words are in its buffer
        read(slot, 0, nxt);
    }
    place_code();
    steps<64, 80>(R, H, c, own, cur, nxt);
    uint64_t at80[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) at80[i] = R[i];
    step<80>(R, c, own, 1);
    step<81>(R, c, own, 1);
#undef HV_PIN
    if (b < nblk) {
        H[0] += at80[0];
        H[1] += at80[1];
        H[2] += c.m ? R[2] : at80[2];
        H[3] += c.m ? R[3] : at80[3];
    }
}

__global__ void __launch_bounds__(256) sha384_chain_kernel(const LeafDesc* __restrict__ desc, uint64_t n_slots,
                                                           uint64_t out_bound, uint8_t* __restrict__ digests) {
    __shared__ uint4 sched[3][kEntries][kRow];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t base = (uint64_t)blockIdx.x * 64;
    // every wave holds the 64 descriptors once, for the block counts
    uint64_t slot = base + lane;
    bool live = slot < n_slots;
    LeafDesc d = {0, 0, 0};
    if (live) d = desc[slot];
    uint32_t nfull = (uint32_t)(d.nbytes >> 7), r = (uint32_t)(d.nbytes & 127);
    uint32_t nblk = live ? nfull + (r <= 111 ? 1u : 2u) : 0u;
    uint32_t nmax = nblk;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t x = __shfl_xor(nmax, o);
        nmax = x > nmax ? x : nmax;
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);

    if (wave >= 2) {
        const uint32_t p = wave & 1;
        // the ones, each producer's half of them before barrier 1
        if (lane < 60) sched[(60 * p + lane) / kEntries][(60 * p + lane) % kEntries][64] = make_uint4(1, 0, 1, 0);
        if (__all((d.src & 15) == 0))
            produce_alternate<true>(p, d.src, d.nbytes, nfull, r, nblk, nmax, lane, sched);
        else
            produce_alternate<false>(p, d.src, d.nbytes, nfull, r, nblk, nmax, lane, sched);
        return;
    }
    const uint32_t chunk = 32 * wave + (lane >> 1);
    slot = base + chunk;
    live = slot < n_slots;
    d = {0, 0, 0};
    if (live) d = desc[slot];
    nfull = (uint32_t)(d.nbytes >> 7);
    r = (uint32_t)(d.nbytes & 127);
    nblk = live ? nfull + (r <= 111 ? 1u : 2u) : 0u;
    const bool e = lane & 1;
    const Half c = {e ? 4u : 6u, e ? 27u : 11u, e ? 14u : 28u, e ? 0u : ~0u};
    uint64_t H[4] = {e ? kInit384[4] : kInit384[2], e ? kInit384[5] : kInit384[3], e ? kInit384[6] : kInit384[0],
                     e ? kInit384[7] : kInit384[1]};
    const uint32_t col = e ? chunk : 64u;
    uint4 A[8], B[8];  // five groups per block: the sets' roles swap from block to block
    if (nmax > 0) {
        lds_barrier();
        lds_barrier();  // block 0's words are in buffer 0
#pragma unroll
        for (int g = 0; g < 8; ++g) A[g] = sched[0][g][col];
    }
    uint32_t buf = 0;  // b % 3
    for (uint32_t b = 0; b < nmax; b += 2) {
        consume(b, buf, nmax, nblk, col, sched, H, c, A, B);
        if (b + 1 < nmax) consume(b + 1, buf, nmax, nblk, col, sched, H, c, B, A);
    }
    if (live && d.out < out_bound) {
        // H0..H3 from the a lane, H4 and H5 from the e lane
        uint4* out = reinterpret_cast<uint4*>(digests + 48 * d.out);
        const uint4 first = make_uint4(__builtin_bswap32(hi32(H[0])), __builtin_bswap32(lo32(H[0])),
                                       __builtin_bswap32(hi32(H[1])), __builtin_bswap32(lo32(H[1])));
        const uint4 second = make_uint4(__builtin_bswap32(hi32(H[2])), __builtin_bswap32(lo32(H[2])),
                                        __builtin_bswap32(hi32(H[3])), __builtin_bswap32(lo32(H[3])));
        if (e) {
            out[2] = first;
        } else {
            out[0] = second;
            out[1] = first;
        }
    }
}

}  // namespace

hipError_t launch_sha384_auto(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              hipStream_t s, bool background) {
    const int k = leaf_launch_for(kAlgSha384, n_slots, background, device_cus());
    if (k == kLeafOneWave) return launch_sha384_leaves(desc, n_slots, out_bound, digests, s);
    return launch_sha384_split(desc, n_slots, out_bound, digests, k == kLeafTwoWaveCompact, s);
}

hipError_t launch_sha384_split(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                               bool two_pairs, hipStream_t s) {
    for (uint64_t base = 0; base < n_slots; base += kMaxSlotsPerLaunch) {
        const uint64_t n = n_slots - base < kMaxSlotsPerLaunch ? n_slots - base : kMaxSlotsPerLaunch;
        if (!two_pairs)
            sha384_chain_kernel<<<(unsigned)((n + 63) / 64), 256, 0, s>>>(desc + base, n, out_bound, digests);
        else
            sha384_pairs_kernel<<<(unsigned)((n + 127) / 128), 256, 0, s>>>(desc + base, n, out_bound, digests);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace hv
