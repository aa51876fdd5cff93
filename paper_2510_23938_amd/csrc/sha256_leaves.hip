// sha256_leaves.hip -- SHA-256 of every chunk (Algorithm 1's per-chunk GPU
// hash), one chunk per lane, 64 chunks per wave.
//
// SHA-256 is a chain of dependent compressions (Merkle-Damgard), so a chunk
// cannot be split across lanes; parallelism is the number of chunks.  Each
// lane keeps the eight state words and a 16-word message-schedule ring in
// VGPRs and runs FIPS 180-4's padding itself (section 5.1.1): whole 64-byte
// blocks first, then one or two final blocks holding the 0..63 tail bytes,
// the 0x80 byte, zeros and the 64-bit bit length.
//
// Load path for whole blocks (16-byte aligned chunks, the usual case): the
// wave stages its 64 chunks through LDS, 128 bytes (two blocks, one HBM line)
// per chunk per stage, with direct-to-LDS 16-byte loads
// (global_load_lds_dwordx4).  Load instruction j of a stage covers chunks
// 8j..8j+7, eight lanes per chunk, so every instruction reads eight whole
// 128-byte lines and every line is read from HBM once.  The 16-byte slots of
// a chunk's row are XOR-swizzled by chunk index so that the 64 lanes reading
// their own rows with ds_read_b128 hit distinct banks.  A stage is copied to
// VGPRs before the next stage's loads are issued into the same buffer, so
// the loads run under the two compressions of the current stage.  A wave with
// a chunk that is not 16-byte aligned stages the aligned bytes around its
// chunks the same way and shifts them into place in registers.
//
// Memory safety at tails: the final partial block is read with aligned dword
// loads that each contain at least one byte of the chunk, so no access
// touches a page the chunk does not touch; bytes past the end are masked off.
#include "balance.h"
#include "hv_kernels.h"
#include "sha256_device.h"
#include "stage.h"

namespace hv {
namespace {

constexpr int kThreads = 256;                     // four waves per workgroup
constexpr int kWaves = kThreads / 64;
constexpr int kRowsPerLoad = 1024 / kStageBytes;  // chunks covered by one 64-lane 16-byte load

// Swizzle of a chunk's 16-byte slots within its LDS row.  Consecutive lanes
// (rows) differ in (c ^ c>>3) & 7, so the eight slots a group of lanes reads
// at once fall in different banks whether the LDS serves 8 or 16 lanes of a
// 16-byte read per cycle.
__device__ __forceinline__ uint32_t swizzle(uint32_t c) { return (c ^ (c >> 3)) & 7u; }

__device__ __forceinline__ void words_from(const uint4& x0, const uint4& x1, const uint4& x2, const uint4& x3,
                                           uint32_t W[16]) {
    W[0] = bswap(x0.x); W[1] = bswap(x0.y); W[2] = bswap(x0.z); W[3] = bswap(x0.w);
    W[4] = bswap(x1.x); W[5] = bswap(x1.y); W[6] = bswap(x1.z); W[7] = bswap(x1.w);
    W[8] = bswap(x2.x); W[9] = bswap(x2.y); W[10] = bswap(x2.z); W[11] = bswap(x2.w);
    W[12] = bswap(x3.x); W[13] = bswap(x3.y); W[14] = bswap(x3.z); W[15] = bswap(x3.w);
}

__device__ __forceinline__ void wait_vm_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)
__device__ __forceinline__ void wait_lgkm_all() { __builtin_amdgcn_s_waitcnt(0xC07F); }  // lgkmcnt(0)

// Whole blocks of the wave's 64 chunks (every lane's chunk 16-byte aligned),
// staged through this wave's 8 KB LDS row buffer.  nfull: this lane's whole
// blocks (at most 2^31 under the library's chunk-size limit, so the block
// counts below cannot wrap; byte offsets take 64 bits).
__device__ __forceinline__ void full_blocks_lds(uint32_t H[8], uint64_t src, uint32_t nfull, uint8_t* rows) {
    uint32_t lane = threadIdx.x & 63;
    // opaque, so that in a kernel that calls this in a loop the addresses
    // derived from it are not kept in registers across the calls
    asm volatile("" : "+v"(lane));
    uint32_t nmax = nfull, nmin = nfull;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t a = __shfl_xor(nmax, o), b = __shfl_xor(nmin, o);
        nmax = a > nmax ? a : nmax;
        nmin = b < nmin ? b : nmin;
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);
    nmin = __builtin_amdgcn_readfirstlane(nmin);
    const uint32_t stages = (nmax + 1) / 2;
    if (stages == 0) return;

    // The 16 bytes this lane moves for load j of every stage: chunk 8j + lane/8,
    // source slot (lane % 8) ^ swizzle(chunk), landing in LDS slot lane % 8.
    const uint8_t* from[kRowsPerLoad];
    uint32_t until[kRowsPerLoad];  // stages in which that slot lies in a whole block
#pragma unroll
    for (int j = 0; j < kRowsPerLoad; ++j) {
        const uint32_t c = kRowsPerLoad * j + (lane >> 3);
        const uint32_t slot = (lane & 7) ^ swizzle(c);
        const uint64_t s = __shfl(src, (int)c);
        const uint32_t nf = __shfl(nfull, (int)c);
        from[j] = reinterpret_cast<const uint8_t*>(s) + 16 * slot;
        until[j] = slot < 4 ? (nf + 1) / 2 : nf / 2;
    }
    const bool uniform = nmin == nmax;

#pragma unroll
    for (int j = 0; j < kRowsPerLoad; ++j)
        if (0 < until[j]) __builtin_amdgcn_global_load_lds(from[j], rows + 1024 * j, 16, 0, 0);

    const uint8_t* row = rows + kStageBytes * lane;
    const uint32_t sw = swizzle(lane);
    for (uint32_t st = 0; st < stages; ++st) {
        wait_vm_all();  // stage st is in LDS
        uint4 r[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) r[k] = *reinterpret_cast<const uint4*>(row + 16 * (k ^ sw));
        wait_lgkm_all();  // and in VGPRs: the buffer may be refilled
        const uint32_t nx = st + 1;
        if (nx < stages) {
            const uint64_t off = stage_offset(nx);
            if (uniform && 2 * nx + 1 < nmax) {  // whole stage valid for every chunk
#pragma unroll
                for (int j = 0; j < kRowsPerLoad; ++j)
                    __builtin_amdgcn_global_load_lds(from[j] + off, rows + 1024 * j, 16, 0, 0);
            } else {
#pragma unroll
                for (int j = 0; j < kRowsPerLoad; ++j)
                    if (nx < until[j]) __builtin_amdgcn_global_load_lds(from[j] + off, rows + 1024 * j, 16, 0, 0);
            }
        }
        uint32_t W[16];
        if (2 * st < nfull) {
            words_from(r[0], r[1], r[2], r[3], W);
            compress(H, W);
        }
        if (2 * st + 1 < nfull) {
            words_from(r[4], r[5], r[6], r[7], W);
            compress(H, W);
        }
    }
}

// Up to 64 bytes starting at p (any alignment) as 16 little-endian words of
// the bytes p[0..63]; bytes at or past `valid` are undefined.  Loads only the
// aligned dwords that hold at least one of the first `valid` bytes.
__device__ __forceinline__ void gather_words(const uint8_t* p, uint32_t valid, uint32_t X[16]) {
    const uintptr_t pa = reinterpret_cast<uintptr_t>(p);
    const uint32_t sh = (uint32_t)(pa & 3);
    const uint32_t* a = reinterpret_cast<const uint32_t*>(pa - sh);
    uint32_t D[17];
    const uint32_t end = valid > 0 ? sh + valid : 0u;  // no bytes: no loads, whatever the address
#pragma unroll
    for (int k = 0; k < 17; ++k) D[k] = (uint32_t)(4 * k) < end ? a[k] : 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) X[i] = __builtin_amdgcn_alignbyte(D[i + 1], D[i], sh);
}

// One block's 16 message words from the 20 dwords D in which it starts `shift`
// = 0..15 bytes in: two rounds of masked selects for whole dwords, and one byte
// permute per word that also puts the bytes in order (sel).
__device__ __forceinline__ void shifted_words(const uint32_t* D, uint32_t by_two, uint32_t by_one, uint32_t sel,
                                              uint32_t W[16]) {
    uint32_t X[18];
#pragma unroll
    for (int i = 0; i < 18; ++i) X[i] = choose(by_two, D[i + 2], D[i]);
#pragma unroll
    for (int i = 0; i < 17; ++i) X[i] = choose(by_one, X[i + 1], X[i]);
#pragma unroll
    for (int i = 0; i < 16; ++i) W[i] = __builtin_amdgcn_perm(X[i + 1], X[i], sel);
}

// Whole blocks of the wave's 64 chunks at any alignment, on the staging of
// full_blocks_lds: a stage is the eight 16-byte granules 8s + 1..8s + 8 of each
// chunk, counted from the granule its first byte lies in, and the last one
// read stays in registers as the first of the next stage.  A granule is loaded
// only if it holds a byte of a whole block.  The realignment adds 35
// operations to a block's 1405 (byte order included in both); a gather of each
// lane's own dwords, 17 loads of 64 lines per block, was bound by those loads
// instead.
__device__ __forceinline__ void full_blocks_any(uint32_t H[8], uint64_t src, uint32_t nfull, uint8_t* rows) {
    uint32_t lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // as in full_blocks_lds
    const uint32_t shift = (uint32_t)src & 15;
    uint4 first = make_uint4(0, 0, 0, 0);
    if (nfull > 0) first = *reinterpret_cast<const uint4*>(src - shift);
    const uint8_t* from[kRowsPerLoad];
    uint32_t until[kRowsPerLoad];  // stages in which that slot holds a byte of a whole block
    uint32_t nmax = nfull, all = 0xffffffffu;
#pragma unroll
    for (int j = 0; j < kRowsPerLoad; ++j) {
        const uint32_t c = kRowsPerLoad * j + (lane >> 3);
        const uint32_t at = 16 * (1 + ((lane & 7) ^ swizzle(c)));
        const uint64_t s = __shfl(src, (int)c);
        const uint64_t end = (s & 15) + 64 * (uint64_t)__shfl(nfull, (int)c);
        from[j] = reinterpret_cast<const uint8_t*>(s & ~(uint64_t)15) + at;
        until[j] = end > at ? (uint32_t)((end - at + kStageBytes - 1) / kStageBytes) : 0u;
        all = until[j] < all ? until[j] : all;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t x = __shfl_xor(nmax, o), y = __shfl_xor(all, o);
        nmax = x > nmax ? x : nmax;
        all = y < all ? y : all;
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);
    all = __builtin_amdgcn_readfirstlane(all);  // stages that every slot of every chunk takes part in
    const uint32_t stages = (nmax + 1) / 2;
    if (stages == 0) return;
#pragma unroll
    for (int j = 0; j < kRowsPerLoad; ++j)
        if (0 < until[j]) __builtin_amdgcn_global_load_lds(from[j], rows + 1024 * j, 16, 0, 0);

    const uint8_t* row = rows + kStageBytes * lane;
    const uint32_t sw = swizzle(lane);
    const uint32_t by_two = shift & 8 ? ~0u : 0u, by_one = shift & 4 ? ~0u : 0u;
    const uint32_t sel = 0x00010203u + 0x01010101u * (shift & 3);
    for (uint32_t st = 0; st < stages; ++st) {
        wait_vm_all();  // stage st is in LDS
        uint32_t D[36] = {first.x, first.y, first.z, first.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint4 r = *reinterpret_cast<const uint4*>(row + 16 * (k ^ sw));
            D[4 + 4 * k] = r.x; D[5 + 4 * k] = r.y; D[6 + 4 * k] = r.z; D[7 + 4 * k] = r.w;
        }
        wait_lgkm_all();  // and in VGPRs: the buffer may be refilled
        first = make_uint4(D[32], D[33], D[34], D[35]);
        const uint32_t nx = st + 1;
        if (nx < stages) {
            const uint64_t off = stage_offset(nx);
            if (nx < all) {
#pragma unroll
                for (int j = 0; j < kRowsPerLoad; ++j)
                    __builtin_amdgcn_global_load_lds(from[j] + off, rows + 1024 * j, 16, 0, 0);
            } else {
#pragma unroll
                for (int j = 0; j < kRowsPerLoad; ++j)
                    if (nx < until[j]) __builtin_amdgcn_global_load_lds(from[j] + off, rows + 1024 * j, 16, 0, 0);
            }
        }
        uint32_t W[16];
        if (2 * st < nfull) {
            shifted_words(D, by_two, by_one, sel, W);
            compress(H, W);
        }
        if (2 * st + 1 < nfull) {
            shifted_words(D + 16, by_two, by_one, sel, W);
            compress(H, W);
        }
    }
}

// Final block(s): r = 0..63 tail bytes at p, then 0x80, zeros and the bit
// length of the whole chunk (total bytes).
__device__ __forceinline__ void final_blocks(uint32_t H[8], const uint8_t* p, uint32_t r, uint64_t total) {
    uint32_t W[16];
    gather_words(p, r, W);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int nv = (int)r - 4 * i;  // tail bytes that fall in word i
        const uint32_t keep = nv >= 4 ? 0xffffffffu : (nv <= 0 ? 0u : (1u << (8 * nv)) - 1u);
        const uint32_t pad = (nv >= 0 && nv < 4) ? (0x80u << (8 * nv)) : 0u;
        W[i] = bswap((W[i] & keep) | pad);
    }
    const uint64_t bits = total * 8;
    if (r <= 55) {
        W[14] = (uint32_t)(bits >> 32);
        W[15] = (uint32_t)bits;
        compress(H, W);
    } else {
        compress(H, W);
#pragma unroll
        for (int i = 0; i < 14; ++i) W[i] = 0;
        W[14] = (uint32_t)(bits >> 32);
        W[15] = (uint32_t)bits;
        compress(H, W);
    }
}

// The whole blocks among blocks [from, to) of a wave's 64 chunks, one per lane;
// with `last`, all from `from` on.
__device__ __forceinline__ void whole_blocks(uint32_t H[8], const LeafDesc& d, uint32_t from, uint32_t to, bool last,
                                             uint8_t* rows) {
    const uint32_t nfull = (uint32_t)(d.nbytes >> 6);
    const uint32_t f0 = from < nfull ? from : nfull, f1 = last || to > nfull ? nfull : to;
    if (__all((d.src & 15) == 0))
        full_blocks_lds(H, d.src + ((uint64_t)f0 << 6), f1 - f0, rows);
    else
        full_blocks_any(H, d.src + ((uint64_t)f0 << 6), f1 - f0, rows);
}

// The rest of a wave's chunks, and their digests.
__device__ __forceinline__ void finish(uint32_t H[8], const LeafDesc& d, bool live, uint64_t out_bound,
                                       uint8_t* digests) {
    const uint64_t whole = d.nbytes & ~(uint64_t)63;
    final_blocks(H, reinterpret_cast<const uint8_t*>(d.src) + whole, (uint32_t)(d.nbytes & 63), d.nbytes);
    if (live && d.out < out_bound) store_digest(digests + 32 * d.out, H);
}

__device__ __forceinline__ LeafDesc load_desc(const LeafDesc* __restrict__ desc, uint64_t slot, uint64_t n_slots) {
    LeafDesc d = {0, 0, 0};
    if (slot < n_slots) d = desc[slot];
    return d;
}

__global__ void __launch_bounds__(kThreads) sha256_leaves_kernel(const LeafDesc* __restrict__ desc, uint64_t n_slots,
                                                                 uint64_t out_bound, uint8_t* __restrict__ digests) {
    __shared__ __attribute__((aligned(16))) uint8_t stage[kWaves][64 * kStageBytes];
    const uint64_t slot = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    const LeafDesc d = load_desc(desc, slot, n_slots);
    uint32_t H[8];
    init_state(H);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    whole_blocks(H, d, 0, 0, true, stage[wave]);
    finish(H, d, slot < n_slots, out_bound, digests);
}

// The same over the intervals of a tape (balance.h), one per wave.
__global__ void __launch_bounds__(kThreads, 3) sha256_tape_kernel(const LeafDesc* __restrict__ desc, uint64_t n_slots,
                                                                  uint64_t out_bound, uint8_t* __restrict__ digests,
                                                                  const Tape tape) {
    __shared__ __attribute__((aligned(16))) uint8_t stage[kWaves][64 * kStageBytes];
    const uint32_t in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wave = blockIdx.x * kWaves + in_block;
    TapeWalk walk(tape, n_slots, wave);
    Piece piece;
    while (walk.next(&piece)) {
        uint32_t lane = threadIdx.x & 63;
        uint32_t H[8];
        if (piece.from > 0 && !load_states<8>(tape, wave, H)) piece.from = 0;
        if (piece.from == 0) init_state(H);
        whole_blocks(H, load_desc(desc, 64 * piece.group + lane, n_slots), piece.from, piece.to, piece.last,
                     stage[in_block]);
        if (piece.last) {
            // read again: kept across the blocks, the descriptor's registers
            // would cost the third wave per SIMD
            asm volatile("" : "+v"(lane));
            const uint64_t slot = 64 * piece.group + lane;
            finish(H, load_desc(desc, slot, n_slots), slot < n_slots, out_bound, digests);
        } else {
            save_states<8>(tape, wave, H);
        }
    }
}

}  // namespace

hipError_t launch_sha256_tape(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              const Tape& tape, hipStream_t s) {
    sha256_tape_kernel<<<tape.waves / kWaves, kThreads, 0, s>>>(desc, n_slots, out_bound, digests, tape);
    return hipGetLastError();
}

hipError_t launch_sha256_leaves(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                                hipStream_t s) {
    for (uint64_t base = 0; base < n_slots; base += kMaxSlotsPerLaunch) {
        const uint64_t n = n_slots - base < kMaxSlotsPerLaunch ? n_slots - base : kMaxSlotsPerLaunch;
        sha256_leaves_kernel<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(desc + base, n, out_bound,
                                                                                          digests);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace hv
