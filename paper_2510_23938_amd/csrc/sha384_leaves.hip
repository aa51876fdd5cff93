// sha384_leaves.hip -- SHA-384 of every chunk (FIPS 180-4 section 6.5), one
// chunk per lane, 64 chunks per wave: the hash of the paper's own kernel
// listings, on the same schedule and load path as the SHA-256 leaf kernel.
//
// Blocks are 128 bytes, so one LDS stage -- 128 bytes per chunk, eight
// 16-byte direct-to-LDS loads per wave, swizzled rows -- is exactly one block.
// Padding (section 5.1.2): the 0..127 tail bytes, 0x80, zeros and the 128-bit
// big-endian bit length, in one final block when the tail is at most 111
// bytes, else two.  Tail reads are aligned dwords that each hold at least one
// chunk byte, as in the SHA-256 kernel.
#include "balance.h"
#include "hv_kernels.h"
#include "sha384_device.h"
#include "stage.h"

namespace hv {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kRowsPerLoad = 1024 / kStageBytes;

__device__ __forceinline__ uint32_t swizzle(uint32_t c) { return (c ^ (c >> 3)) & 7u; }
__device__ __forceinline__ void wait_vm_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)
__device__ __forceinline__ void wait_lgkm_all() { __builtin_amdgcn_s_waitcnt(0xC07F); }  // lgkmcnt(0)

__device__ __forceinline__ void block_from(const uint4 r[8], uint64_t W[16]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        W[2 * k] = be64(r[k].x, r[k].y);
        W[2 * k + 1] = be64(r[k].z, r[k].w);
    }
}

// Whole 128-byte blocks of the wave's 64 chunks (all 16-byte aligned), staged
// through this wave's 8 KB LDS rows; nfull <= 2^30 (the chunk-size limit).
__device__ __forceinline__ void full_blocks_lds(uint64_t H[8], uint64_t src, uint32_t nfull, uint8_t* rows) {
    uint32_t lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // as in the SHA-256 kernel
    uint32_t nmax = nfull, nmin = nfull;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t a = __shfl_xor(nmax, o), b = __shfl_xor(nmin, o);
        nmax = a > nmax ? a : nmax;
        nmin = b < nmin ? b : nmin;
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);
    nmin = __builtin_amdgcn_readfirstlane(nmin);
    if (nmax == 0) return;

    const uint8_t* from[kRowsPerLoad];
    uint32_t until[kRowsPerLoad];  // blocks of the chunk this lane's slot j belongs to
#pragma unroll
    for (int j = 0; j < kRowsPerLoad; ++j) {
        const uint32_t c = kRowsPerLoad * j + (lane >> 3);
        const uint32_t slot = (lane & 7) ^ swizzle(c);
        const uint64_t s = __shfl(src, (int)c);
        from[j] = reinterpret_cast<const uint8_t*>(s) + 16 * slot;
        until[j] = __shfl(nfull, (int)c);
    }
    const bool uniform = nmin == nmax;

#pragma unroll
    for (int j = 0; j < kRowsPerLoad; ++j)
        if (0 < until[j]) __builtin_amdgcn_global_load_lds(from[j], rows + 1024 * j, 16, 0, 0);

    const uint8_t* row = rows + kStageBytes * lane;
    const uint32_t sw = swizzle(lane);
    for (uint32_t b = 0; b < nmax; ++b) {
        wait_vm_all();
        uint4 r[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) r[k] = *reinterpret_cast<const uint4*>(row + 16 * (k ^ sw));
        wait_lgkm_all();
        const uint32_t nx = b + 1;
        if (nx < nmax) {
            const uint64_t off = stage_offset(nx);
            if (uniform) {
#pragma unroll
                for (int j = 0; j < kRowsPerLoad; ++j)
                    __builtin_amdgcn_global_load_lds(from[j] + off, rows + 1024 * j, 16, 0, 0);
            } else {
#pragma unroll
                for (int j = 0; j < kRowsPerLoad; ++j)
                    if (nx < until[j]) __builtin_amdgcn_global_load_lds(from[j] + off, rows + 1024 * j, 16, 0, 0);
            }
        }
        if (b < nfull) {
            uint64_t W[16];
            block_from(r, W);
            compress512(H, W);
        }
    }
}

// Up to 128 bytes at p (any alignment) as 32 little-endian words; bytes at or
// past `valid` are undefined.  Loads only aligned dwords holding a valid byte.
__device__ __forceinline__ void gather_words(const uint8_t* p, uint32_t valid, uint32_t X[32]) {
    const uintptr_t pa = reinterpret_cast<uintptr_t>(p);
    const uint32_t sh = (uint32_t)(pa & 3);
    const uint32_t* a = reinterpret_cast<const uint32_t*>(pa - sh);
    uint32_t D[33];
    const uint32_t end = valid > 0 ? sh + valid : 0u;  // no bytes: no loads, whatever the address
#pragma unroll
    for (int k = 0; k < 33; ++k) D[k] = (uint32_t)(4 * k) < end ? a[k] : 0u;
#pragma unroll
    for (int i = 0; i < 32; ++i) X[i] = __builtin_amdgcn_alignbyte(D[i + 1], D[i], sh);
}

// Whole blocks of the wave's 64 chunks at any alignment, as in the SHA-256
// kernel: a stage is the granules 8b + 1..8b + 8 of each chunk, the last one
// read starts the next block, and selects and byte permutes shift the words
// into place (67 operations more than a block's 3426).
__device__ __forceinline__ void full_blocks_any(uint64_t H[8], uint64_t src, uint32_t nfull, uint8_t* rows) {
    uint32_t lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
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
        const uint64_t end = (s & 15) + 128 * (uint64_t)__shfl(nfull, (int)c);
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
    if (nmax == 0) return;
#pragma unroll
    for (int j = 0; j < kRowsPerLoad; ++j)
        if (0 < until[j]) __builtin_amdgcn_global_load_lds(from[j], rows + 1024 * j, 16, 0, 0);

    const uint8_t* row = rows + kStageBytes * lane;
    const uint32_t sw = swizzle(lane);
    const uint32_t by_two = shift & 8 ? ~0u : 0u, by_one = shift & 4 ? ~0u : 0u;
    const uint32_t sel = 0x00010203u + 0x01010101u * (shift & 3);
    for (uint32_t b = 0; b < nmax; ++b) {
        wait_vm_all();
        uint32_t D[36] = {first.x, first.y, first.z, first.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint4 r = *reinterpret_cast<const uint4*>(row + 16 * (k ^ sw));
            D[4 + 4 * k] = r.x; D[5 + 4 * k] = r.y; D[6 + 4 * k] = r.z; D[7 + 4 * k] = r.w;
        }
        wait_lgkm_all();
        first = make_uint4(D[32], D[33], D[34], D[35]);
        const uint32_t nx = b + 1;
        if (nx < nmax) {
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
        if (b < nfull) {
#pragma unroll
            for (int i = 0; i < 34; ++i) D[i] = __builtin_amdgcn_bitop3_b32(by_two, D[i + 2], D[i], 0xCA);
#pragma unroll
            for (int i = 0; i < 33; ++i) D[i] = __builtin_amdgcn_bitop3_b32(by_one, D[i + 1], D[i], 0xCA);
            uint64_t W[16];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                W[i] = pack(__builtin_amdgcn_perm(D[2 * i + 1], D[2 * i], sel),
                            __builtin_amdgcn_perm(D[2 * i + 2], D[2 * i + 1], sel));
            compress512(H, W);
        }
    }
}

// Final block(s): r = 0..127 tail bytes at p, 0x80, zeros, 128-bit bit length.
__device__ __forceinline__ void final_blocks(uint64_t H[8], const uint8_t* p, uint32_t r, uint64_t total) {
    uint32_t X[32];
    gather_words(p, r, X);
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const int nv = (int)r - 4 * i;
        const uint32_t keep = nv >= 4 ? 0xffffffffu : (nv <= 0 ? 0u : (1u << (8 * nv)) - 1u);
        const uint32_t pad = (nv >= 0 && nv < 4) ? (0x80u << (8 * nv)) : 0u;
        X[i] = (X[i] & keep) | pad;
    }
    uint64_t W[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) W[i] = be64(X[2 * i], X[2 * i + 1]);
    const uint64_t bits_hi = total >> 61, bits_lo = total << 3;
    if (r <= 111) {
        W[14] = bits_hi;
        W[15] = bits_lo;
        compress512(H, W);
    } else {
        compress512(H, W);
#pragma unroll
        for (int i = 0; i < 14; ++i) W[i] = 0;
        W[14] = bits_hi;
        W[15] = bits_lo;
        compress512(H, W);
    }
}

// Blocks [from, to) of a wave's 64 chunks, as in the SHA-256 kernel.
__device__ __forceinline__ void hash_blocks(uint64_t H[8], const LeafDesc& d, uint32_t from, uint32_t to, bool last,
                                            uint8_t* rows) {
    const uint8_t* p = reinterpret_cast<const uint8_t*>(d.src);
    const uint32_t nfull = (uint32_t)(d.nbytes >> 7);
    const uint32_t f0 = from < nfull ? from : nfull, f1 = last || to > nfull ? nfull : to;
    if (__all((d.src & 15) == 0))
        full_blocks_lds(H, d.src + ((uint64_t)f0 << 7), f1 - f0, rows);
    else
        full_blocks_any(H, d.src + ((uint64_t)f0 << 7), f1 - f0, rows);
    if (last) final_blocks(H, p + ((uint64_t)nfull << 7), (uint32_t)(d.nbytes & 127), d.nbytes);
}

__global__ void __launch_bounds__(kThreads) sha384_leaves_kernel(const LeafDesc* __restrict__ desc, uint64_t n_slots,
                                                                 uint64_t out_bound, uint8_t* __restrict__ digests) {
    __shared__ __attribute__((aligned(16))) uint8_t stage[kWaves][64 * kStageBytes];
    const uint64_t slot = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool live = slot < n_slots;
    LeafDesc d = {0, 0, 0};
    if (live) d = desc[slot];
    uint64_t H[8];
    init_state384(H);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    hash_blocks(H, d, 0, 0, true, stage[wave]);
    if (live && d.out < out_bound) store_digest384(digests + 48 * d.out, H);
}

// The same over the intervals of a tape (balance.h), one per wave.
__global__ void __launch_bounds__(kThreads, 3) sha384_tape_kernel(const LeafDesc* __restrict__ desc, uint64_t n_slots,
                                                                  uint64_t out_bound, uint8_t* __restrict__ digests,
                                                                  const Tape tape) {
    __shared__ __attribute__((aligned(16))) uint8_t stage[kWaves][64 * kStageBytes];
    const uint32_t in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wave = blockIdx.x * kWaves + in_block;
    TapeWalk walk(tape, n_slots, wave);
    Piece piece;
    while (walk.next(&piece)) {
        const uint64_t slot = 64 * piece.group + (threadIdx.x & 63);
        LeafDesc d = {0, 0, 0};
        if (slot < n_slots) d = desc[slot];
        uint64_t H[8];
        uint32_t words[16];
        if (piece.from > 0 && !load_states<16>(tape, wave, words)) piece.from = 0;
        if (piece.from == 0) {
            init_state384(H);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) H[i] = pack(words[2 * i + 1], words[2 * i]);
        }
        hash_blocks(H, d, piece.from, piece.to, piece.last, stage[in_block]);
        if (!piece.last) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                words[2 * i] = lo32(H[i]);
                words[2 * i + 1] = hi32(H[i]);
            }
            save_states<16>(tape, wave, words);
        } else if (slot < n_slots && d.out < out_bound) {
            store_digest384(digests + 48 * d.out, H);
        }
    }
}

}  // namespace

hipError_t launch_sha384_tape(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                              const Tape& t, hipStream_t s) {
    sha384_tape_kernel<<<t.waves / kWaves, kThreads, 0, s>>>(desc, n_slots, out_bound, digests, t);
    return hipGetLastError();
}

hipError_t launch_sha384_leaves(const LeafDesc* desc, uint64_t n_slots, uint64_t out_bound, uint8_t* digests,
                                hipStream_t s) {
    for (uint64_t base = 0; base < n_slots; base += kMaxSlotsPerLaunch) {
        const uint64_t n = n_slots - base < kMaxSlotsPerLaunch ? n_slots - base : kMaxSlotsPerLaunch;
        sha384_leaves_kernel<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(desc + base, n, out_bound,
                                                                                          digests);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace hv
