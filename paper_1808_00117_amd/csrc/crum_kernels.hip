// HIP kernels of the incremental snapshot (gfx950, wave64).
//
// Snapshot pipeline (k_begin once a call, then one launch of each per chunk of
// the page space, or per group of requests of a plan):
//   k_begin   tables from pinned memory into scratch.
//   k_diff    per diff unit (min(page, 4-16 KiB)): OR over 16-byte words of
//             (cur ^ shadow) != 0, read with coalesced 128-bit loads and
//             reduced across the wave by ballot; one flag byte per unit.
//   k_bitmap  per 64 pages: OR of each page's unit flags, then one ballot
//             gives the u64 bitmap word (short ranges: inside k_scan).
//   k_scan    one workgroup: exclusive prefix sum of popcount(word) -> slot of
//             each word's first dirty page, continuing a running total so the
//             page space can be processed in chunks; at the end, per-request
//             dirty counts, image offsets and the capacity check.  A short
//             range also gets the k_list step here.
//   k_list    per word: ballot compaction, lane with bit set writes its page
//             index at prefix + popcount(bits below the lane).
//   k_pack    per dirty page (or piece of up to 64 KiB): copy into the
//             image's page area, optionally into the shadow, and CRC-32C on
//             the way; k_finalize combines the piece CRCs of larger pages.
//   k_header  per request, over one or more workgroups: header, region
//             table, bitmap, CRC array, pads, crcs_crc, meta_crc.
// Restore: k_restore_check (the image's own checks, also over one or more
// workgroups), k_scan, k_list, k_pack (verify), k_pack (scatter).
//
// CRC-32C on the device.  The polynomial arithmetic is in gf2.h.  Page bytes go
// through the matrix cores (k_pack): a raw CRC is linear over GF(2), so the 32
// CRC bits of a 4 KiB batch are a 32 x 32768 bit matrix times its bits, and
// the FP4 matrix instruction counts, per CRC bit, the set bits that reach it;
// the count's parity is the bit.  See fold_4k.  The header's two messages (the
// prefix and the CRC array) go the same way.  Pieces of one page, and shares of
// one message, combine by a shift by the bytes that follow them; the standard
// CRC adds crc_init_fix(page bytes).
#include "crum_dev.h"
#include "diff_grid.h"
#include "gf2.h"

#include <algorithm>
#include <cstddef>
#include <cstring>

namespace crum {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Pointers into global memory.  Region and staging pointers reach the kernels
// inside structs or after arithmetic the compiler cannot follow, so it would
// use flat instructions; a flat access counts against the LDS/scalar counter
// as well, so every wait for an LDS table lookup would also wait for each
// load and store in flight.  Casting keeps them global.
typedef const u32x4 __attribute__((address_space(1)))* gcv4;
typedef u32x4 __attribute__((address_space(1)))* gv4;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef const u32x2 __attribute__((address_space(1)))* gcv2;
typedef u32x2 __attribute__((address_space(1)))* gv2;
typedef const uint32_t __attribute__((address_space(1)))* gcu32;
typedef uint32_t __attribute__((address_space(1)))* gu32;

// ------------------------------------------------------------ CRC tables

static void fill_crc_tables(CrcTables* h)
{
    const uint32_t x4k = gf2_xpow8n(4096);
    for (int i = 0; i < 4; ++i)
        for (int b = 0; b < 256; ++b)
            h->z4k[i][b] = gf2_mulmod((uint32_t)b << (8 * i), x4k);
    for (int i = 0; i < 64; ++i)
        h->xp[i] = gf2_xpow8n(1ull << i);
    for (int i = 0; i < 31; ++i)
        h->init_fix[i] = crc_init_fix(1ull << i);
    const uint32_t x4 = gf2_xpow8n(4);
    h->xr[0] = 0x80000000u;  // x^0
    for (int i = 1; i < 1024; ++i)
        h->xr[i] = gf2_mulmod(h->xr[i - 1], x4);
    for (int k = 0; k < 3; ++k) {
        const uint32_t x = gf2_xpow8n(4096ull << (8 * k));
        h->xb[k][0] = 0x80000000u;
        for (int i = 1; i < 256; ++i)
            h->xb[k][i] = gf2_mulmod(h->xb[k][i - 1], x);
    }
    // fold_4k's matrix: the CRC bit of matrix row r, and what each data bit adds
    // to it (see there for the layout)
    static const uint32_t unit[4] = {4, 2, 1, 4};  // FP4 2.0, 1.0, 0.5, 2.0
    std::memset(h->mf, 0, sizeof(h->mf));
    for (int step = 0; step < 4; ++step)
        for (int half = 0; half < 2; ++half)
            for (int d = 0; d < 4; ++d) {
                const uint32_t x = gf2_xpow8n(16 - 4 * d + 512 * (7 - (2 * step + half)));
                for (int bit = 0; bit < 32; ++bit) {
                    const uint32_t c = gf2_mulmod(1u << bit, x);
                    const int n = bit >> 2, plane = bit & 3;
                    for (int r = 0; r < 32; ++r) {
                        const int crc_bit = 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3);
                        if ((c >> crc_bit) & 1u)
                            h->mf[step * 4 + plane][32 * half + r][d] |= unit[plane] << (4 * n);
                    }
                }
            }
    for (int j = 0; j < 32; ++j) {
        const uint32_t x = gf2_xpow8n(16 * (31 - j));
        for (int k = 0; k < 8; ++k)
            for (int n = 0; n < 16; ++n)
                h->col[k][n][j] = gf2_mulmod((uint32_t)n << (4 * k), x);
    }
}

// Filled at the first use: every context uploads the same constants.
const CrcTables& crc_tables()
{
    static const CrcTables* t = [] {
        CrcTables* h = new CrcTables;
        fill_crc_tables(h);
        return h;
    }();
    return *t;
}

// LDS layout of the kernels that compute CRCs (words): the column tables (col),
// then the shift-by-4-KiB byte tables (z4k); 20 KiB.
constexpr int kColWords = 8 * 16 * 32;
constexpr int kCrcLdsWords = kColWords + 4 * 256;

// Every kernel of this file runs 256-thread workgroups.
constexpr int kBlock = 256;

// Copy WORDS 4-byte words (16-byte aligned at both ends) from global memory
// into LDS: each thread issues all of its 16-byte loads before its first LDS
// store.  A word-per-iteration loop waits for every load in turn, which cost
// each workgroup tens of memory round trips before its first useful step.
template <int WORDS>
__device__ __forceinline__ void stage_words(uint32_t* __restrict__ dst,
                                            const uint32_t* __restrict__ src)
{
    static_assert(WORDS % 4 == 0, "whole 16-byte vectors");
    constexpr int V = WORDS / 4;
    constexpr int N = (V + kBlock - 1) / kBlock;
    const uint4* s = reinterpret_cast<const uint4*>(src);
    uint4* d = reinterpret_cast<uint4*>(dst);
    uint4 v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int i = (int)threadIdx.x + kBlock * k;
        if (V % kBlock == 0 || i < V)
            v[k] = s[i];
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int i = (int)threadIdx.x + kBlock * k;
        if (V % kBlock == 0 || i < V)
            d[i] = v[k];
    }
}

__device__ __forceinline__ void load_crc_tables(uint32_t* lds, const CrcTables* tabs)
{
    stage_words<kColWords>(lds, &tabs->col[0][0][0]);
    stage_words<4 * 256>(lds + kColWords, &tabs->z4k[0][0]);
    __syncthreads();
}

// LDS word at byte offset `off` (a multiple of 4)
__device__ __forceinline__ uint32_t lds_at(const uint32_t* __restrict__ L, uint32_t off)
{
    return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(L) + off);
}

// a ^ b ^ c in one instruction
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// ------------------------------------------------------------ matrix-core CRC

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// The constant operands of fold_4k: per 1 KiB step and bit plane, this lane's
// 32 FP4 values of the matrix (64 registers for the life of the kernel).
struct CrcMatrix {
    u32x4 a[16];
};

__device__ __forceinline__ void load_crc_matrix(CrcMatrix& m, const CrcTables* __restrict__ tabs,
                                                uint32_t lane)
{
#pragma unroll
    for (int i = 0; i < 16; ++i)
        m.a[i] = *(gcv4)(&tabs->mf[i][lane][0]);
}

__device__ __forceinline__ f32x16 mfma_fp4(u32x4 a, u32x4 b, f32x16 c)
{
    const i32x8 A = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const i32x8 B = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A, B, c, 4, 4, 0, 0, 0, 0);
}

// Raw CRCs of a 4 KiB batch by columns.  w[t]: this lane's 16 bytes of 1 KiB
// step t (word 64t + lane).  Matrix column j = lane % 32 takes the eight words
// j, j + 32, ... , j + 224; lane half h = lane / 32 holds every second one.
// Masking a word with 0x11111111, 0x22222222 and 0x44444444 leaves nibbles
// that are FP4 numbers, 0 or 0.5, 1 or 2, one per data bit (bit 3 of a nibble is
// FP4's sign, so that plane is shifted down to 0.5 first); the matrix holds
// the reciprocal where the bit reaches the CRC bit of the row and 0
// elsewhere.  Every product is then 0 or 1 and every sum a whole number of at
// most 1024: float32 holds them exactly, and their parities are the CRC bits.
// Adding 2^23 puts a count's lowest bit into the lowest bit of the word.  Rows
// are ordered so that the 16 results of a lane of half h are CRC bits 16h ..
// 16h + 15, in order.  Returns those bits in place, zeros elsewhere: the
// column's raw CRC is the XOR of its two lanes.
__device__ __forceinline__ uint32_t fold_4k(const CrcMatrix& m, const u32x4* __restrict__ w,
                                            uint32_t half)
{
    f32x16 c;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        c[i] = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        c = mfma_fp4(m.a[4 * t], w[t] & 0x11111111u, c);
        c = mfma_fp4(m.a[4 * t + 1], w[t] & 0x22222222u, c);
        c = mfma_fp4(m.a[4 * t + 2], w[t] & 0x44444444u, c);
        c = mfma_fp4(m.a[4 * t + 3], (w[t] >> 3) & 0x11111111u, c);
    }
    uint32_t r = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        r = __builtin_amdgcn_alignbit(__float_as_uint(c[i] + 8388608.0f), r, 1);
    return half ? r & 0xFFFF0000u : r >> 16;
}

// The lane's state carried through 4 KiB of zeros.
__device__ __forceinline__ uint32_t shift_4k(const uint32_t* __restrict__ lds, uint32_t s)
{
    return xor3(lds_at(lds, 4u * kColWords + ((s << 2) & 0x3FCu)),
                lds_at(lds, 4u * (kColWords + 256) + ((s >> 6) & 0x3FCu)),
                lds_at(lds, 4u * (kColWords + 512) + ((s >> 14) & 0x3FCu))) ^
           lds_at(lds, 4u * (kColWords + 768) + ((s >> 22) & 0x3FCu));
}

// Raw CRC of the piece from the lanes' column states: column j is followed by
// 31 - j more words, so its state is multiplied by x^(128(31-j)) (eight nibble
// lookups in the column's own tables, one bank per lane) and all lanes are
// XORed.  Uniform over the wave.
__device__ __forceinline__ uint32_t columns_crc(const uint32_t* __restrict__ lds, uint32_t s,
                                                uint32_t lane)
{
    const uint32_t j4 = (lane & 31u) * 4u;
    uint32_t v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t n = k == 0 ? s << 7 : k == 1 ? s << 3 : s >> (4 * k - 7);
        v[k] = lds_at(lds, 2048u * k + ((n & 0x780u) | j4));
    }
    uint32_t r = xor3(xor3(v[0], v[1], v[2]), xor3(v[3], v[4], v[5]), v[6] ^ v[7]);
    // lanes of each row of 16: xor 1, xor 2, then mirrored halves and rows
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0xB1, 0xF, 0xF, true);
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0x4E, 0xF, 0xF, true);
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0x141, 0xF, 0xF, true);
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0x140, 0xF, 0xF, true);
    return (uint32_t)__builtin_amdgcn_readlane((int)r, 0) ^
           (uint32_t)__builtin_amdgcn_readlane((int)r, 16) ^
           (uint32_t)__builtin_amdgcn_readlane((int)r, 32) ^
           (uint32_t)__builtin_amdgcn_readlane((int)r, 48);
}

// ------------------------------------------------------------ k_begin

// Copies up to three pieces of whole 8-byte words between pinned host memory and
// the device: a call's region and request tables and counters, an image's header,
// its prefix and CRC array.  With `done` (pinned), stores 1 there once its one
// workgroup's copy is visible to the host.
__global__ __launch_bounds__(256) void k_begin(CopyList list, uint64_t* __restrict__ done)
{
    for (int k = 0; k < 3; ++k) {
        const uint64_t* src = static_cast<const uint64_t*>(list.src[k]);
        uint64_t* dst = static_cast<uint64_t*>(list.dst[k]);
        const uint64_t n = list.bytes[k] / 8;
        for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n;
             i += (uint64_t)gridDim.x * 256)
            dst[i] = src[i];
    }
    if (done) {
        __threadfence_system();
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(done, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

hipError_t launch_begin(const CopyList& list, uint64_t* done, hipStream_t s)
{
    const uint64_t most = std::max(list.bytes[0], std::max(list.bytes[1], list.bytes[2]));
    const uint64_t need = (most / 8 + 255) / 256;
    const unsigned nb = done ? 1u : (unsigned)(need < 1 ? 1 : need < 256 ? need : 256);
    hipLaunchKernelGGL(k_begin, dim3(nb), dim3(256), 0, s, list, done);
    return hipGetLastError();
}

// ------------------------------------------------------------ region lookup

// Last region whose field (3 first_page, 4 first_unit) is <= key.
template <int FIELD>
__device__ __forceinline__ uint32_t find_region(const DevRegion* __restrict__ regs, uint32_t n,
                                                uint64_t key)
{
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        const uint64_t v = FIELD == 3 ? regs[mid].first_page : regs[mid].first_unit;
        if (v <= key)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// ------------------------------------------------------------ k_diff

// OR over the lane's LOADS 16-byte words of (a ^ b), a and b already offset
// by the lane; loads are 1 KiB apart so each one is coalesced across the wave.
// NT marks the loads non-temporal: the streamed bytes are not kept in the
// caches, which stay available to co-running work.
template <int LOADS, bool NT>
__device__ __forceinline__ uint32_t xor_or(gcv4 __restrict__ a, gcv4 __restrict__ b)
{
    u32x4 va[LOADS], vb[LOADS];
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        if (NT) {
            va[j] = __builtin_nontemporal_load(a + j * 64);
            vb[j] = __builtin_nontemporal_load(b + j * 64);
        } else {
            va[j] = a[j * 64];
            vb[j] = b[j * 64];
        }
    }
    u32x4 x = va[0] ^ vb[0];
#pragma unroll
    for (int j = 1; j < LOADS; ++j)
        x |= va[j] ^ vb[j];
    return x.x | x.y | x.z | x.w;
}

// G consecutive 4 KiB units read as one span of G * 4 KiB: 4G loads per
// array in flight per lane, x[k] = OR of (a ^ b) over unit k's four loads.
template <int G, bool NT>
__device__ __forceinline__ void xor_or_group(gcv4 __restrict__ a, gcv4 __restrict__ b,
                                             uint32_t* x)
{
    u32x4 va[4 * G], vb[4 * G];
#pragma unroll
    for (int j = 0; j < 4 * G; ++j) {
        if (NT) {
            va[j] = __builtin_nontemporal_load(a + j * 64);
            vb[j] = __builtin_nontemporal_load(b + j * 64);
        } else {
            va[j] = a[j * 64];
            vb[j] = b[j * 64];
        }
    }
#pragma unroll
    for (int k = 0; k < G; ++k) {
        u32x4 o = va[4 * k] ^ vb[4 * k];
#pragma unroll
        for (int j = 1; j < 4; ++j)
            o |= va[4 * k + j] ^ vb[4 * k + j];
        x[k] = o.x | o.y | o.z | o.w;
    }
}

// The flag of unit u (one wave); the region lookup is cached in r, r_lo, r_hi.
template <bool NT>
__device__ __forceinline__ void diff_unit(const DevRegion* __restrict__ regs, uint32_t n_regs,
                                          uint64_t u, uint8_t* __restrict__ unit_flags,
                                          const uint64_t* __restrict__ cand, uint32_t lane,
                                          uint32_t& r, uint64_t& r_lo, uint64_t& r_hi)
{
    if (u < r_lo || u >= r_hi) {
        r = find_region<4>(regs, n_regs, u);
        r_lo = regs[r].first_unit;
        r_hi = r_lo + (regs[r].len >> regs[r].unit_shift);
    }
    const DevRegion& R = regs[r];
    const uint32_t us = R.unit_shift;
    if (cand && R.shadow != nullptr) {
        const uint64_t g = R.first_page + ((u - R.first_unit) >> (R.page_shift - us));
        if (!((cand[g >> 6] >> (g & 63)) & 1ull)) {
            if (lane == 0)
                unit_flags[u] = 0;
            return;
        }
    }
    uint32_t x = 1;
    if (R.shadow != nullptr) {
        const uint64_t off = (u - R.first_unit) << us;
        const gcv4 a = (gcv4)(R.cur + off) + lane;
        const gcv4 b = (gcv4)(R.shadow + off) + lane;
        x = us == 12 ? xor_or<4, NT>(a, b) : us == 13 ? xor_or<8, NT>(a, b)
                                                      : xor_or<16, NT>(a, b);
    }
    const uint64_t m = __ballot(x != 0);
    if (lane == 0)
        unit_flags[u] = m != 0;
}

// Diff of global units [u0, u1); unit_flags[u] = 1 when any byte of the unit
// differs from the shadow (or the region has none).  G = 1: one wave per
// unit.  G = 2 or 4: one wave per G consecutive units (from u0); G 4 KiB
// units of one region with a shadow, all candidates when a candidate set is
// given, are read as one span of G * 4 KiB, so a wave keeps 4G loads per
// array in flight; other groups are done one unit at a time.
// prio 1..3 raises the waves' issue priority on their compute unit above
// that of co-running kernels' waves (0 leaves it at the default).
// cand (may be null): a bitmap over global pages from host write tracking;
// a page whose bit is clear is known to equal its shadow, so its units are
// flagged clean without reading either copy.
// stamp (may be null): stamp[0] gets the constant-rate wall clock when
// workgroup 0 starts (the first one dispatched), and every workgroup leaves the clock
// of its end as a maximum in one of kStampSlots words, a cache line apart.  They
// need no reset between launches: a later launch's clocks exceed every earlier one's.
// One word for all would serialize the launch it times: 256 MiB of 4 KiB pages took 77 us
// untimed, 98 with one word for the last 4096 workgroups alone, 82 this way, 1 GiB 326,
// 333 and 339 (of 64 KiB pages 325, 330 and 326).
template <bool NT, int G>
__device__ __forceinline__ void diff_units(const DevRegion* __restrict__ regs, uint32_t n_regs,
                                           uint64_t u0, uint64_t u1,
                                           uint8_t* __restrict__ unit_flags, uint32_t prio,
                                           const uint64_t* __restrict__ cand,
                                           uint64_t* __restrict__ stamp)
{
    if (stamp && blockIdx.x == 0 && threadIdx.x == 0)
        stamp[0] = wall_clock64();
    if (prio == 1)
        __builtin_amdgcn_s_setprio(1);
    else if (prio == 2)
        __builtin_amdgcn_s_setprio(2);
    else if (prio >= 3)
        __builtin_amdgcn_s_setprio(3);
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t wave =
        (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t n_waves = (uint64_t)gridDim.x * 4;
    uint32_t r = 0;
    uint64_t r_lo = 1, r_hi = 0;
    if (G == 1) {
        for (uint64_t u = u0 + wave; u < u1; u += n_waves)
            diff_unit<NT>(regs, n_regs, u, unit_flags, cand, lane, r, r_lo, r_hi);
    } else {
        for (uint64_t base = u0 + G * wave; base < u1; base += G * n_waves) {
            const uint64_t end = base + G < u1 ? base + G : u1;
            if (base < r_lo || base >= r_hi) {
                r = find_region<4>(regs, n_regs, base);
                r_lo = regs[r].first_unit;
                r_hi = r_lo + (regs[r].len >> regs[r].unit_shift);
            }
            const DevRegion& R = regs[r];
            bool fused = end == base + G && base + G <= r_hi && R.unit_shift == 12 &&
                         R.shadow != nullptr;
            if (fused && cand) {
                const uint32_t sh = R.page_shift - 12;
                for (uint64_t u = base; u < end; ++u) {
                    const uint64_t g = R.first_page + ((u - R.first_unit) >> sh);
                    fused = fused && ((cand[g >> 6] >> (g & 63)) & 1ull);
                }
            }
            if (fused) {
                const uint64_t off = (base - R.first_unit) << 12;
                uint32_t x[G];
                xor_or_group<G, NT>((gcv4)(R.cur + off) + lane, (gcv4)(R.shadow + off) + lane,
                                    x);
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    const uint64_t m = __ballot(x[k] != 0);
                    if (lane == 0)
                        unit_flags[base + k] = m != 0;
                }
            } else {
                for (uint64_t u = base; u < end; ++u)
                    diff_unit<NT>(regs, n_regs, u, unit_flags, cand, lane, r, r_lo, r_hi);
            }
        }
    }
    if (stamp) {
        __syncthreads();
        if (threadIdx.x == 0)
            atomicMax(reinterpret_cast<unsigned long long*>(
                          stamp + kStampLine * (1 + blockIdx.x % kStampSlots)),
                      (unsigned long long)wall_clock64());
    }
}

template <bool NT, int G>
__global__ __launch_bounds__(256) void k_diff(const DevRegion* __restrict__ regs,
                                              uint32_t n_regs, uint64_t u0, uint64_t u1,
                                              uint8_t* __restrict__ unit_flags, uint32_t prio,
                                              const uint64_t* __restrict__ cand,
                                              uint64_t* __restrict__ stamp)
{
    diff_units<NT, G>(regs, n_regs, u0, u1, unit_flags, prio, cand, stamp);
}

// The diff of a call with few regions: its tables are kernel arguments, and the
// first workgroup stores them (up to the last region) in scratch for the kernels
// behind it.  That saves the k_begin launch (4.5 us of a 45 us snapshot).
template <bool NT, int G>
__global__ __launch_bounds__(256) void k_diff_first(const CallTables t, CallTables* __restrict__ to,
                                                    uint32_t n_regs, uint64_t u1,
                                                    uint8_t* __restrict__ unit_flags,
                                                    uint32_t prio)
{
    if (blockIdx.x == 0) {
        static_assert(sizeof(CallTables) % 16 == 0 && sizeof(CallTables) / 16 <= 256, "one round");
        const u32x4* src = reinterpret_cast<const u32x4*>(&t);
        if (threadIdx.x < (offsetof(CallTables, regs) + n_regs * sizeof(DevRegion)) / 16)
            reinterpret_cast<u32x4*>(to)[threadIdx.x] = src[threadIdx.x];
    }
    diff_units<NT, G>(t.regs, n_regs, 0, u1, unit_flags, prio, nullptr, nullptr);
}

hipError_t launch_diff_first(const CallTables& t, CallTables* to, uint32_t n_regs, uint64_t u1,
                             uint8_t* unit_flags, int blocks, int nontemporal, int prio,
                             hipStream_t s, int group)
{
    if (group != 2 && group != 4)
        group = 1;
    const uint32_t nb = std::max(diff_grid(u1, (uint32_t)group, (uint32_t)blocks), 1u);
#define CRUM_DIFF(NTV, GV)                                                                    \
    hipLaunchKernelGGL((k_diff_first<NTV, GV>), dim3(nb), dim3(256), 0, s,                     \
                       t, to, n_regs, u1, unit_flags, (uint32_t)prio)
    switch ((nontemporal ? 8 : 0) + group) {
    case 1: CRUM_DIFF(false, 1); break;
    case 2: CRUM_DIFF(false, 2); break;
    case 4: CRUM_DIFF(false, 4); break;
    case 9: CRUM_DIFF(true, 1); break;
    case 10: CRUM_DIFF(true, 2); break;
    default: CRUM_DIFF(true, 4); break;
    }
#undef CRUM_DIFF
    return hipGetLastError();
}

hipError_t launch_diff(const DevRegion* regs, uint32_t n_regs, uint64_t u0, uint64_t u1,
                       uint8_t* unit_flags, int blocks, int nontemporal, int prio,
                       hipStream_t s, const uint64_t* cand, uint64_t* stamp, int group)
{
    if (u1 <= u0)
        return hipSuccess;
    if (group != 2 && group != 4)
        group = 1;
    const uint32_t nb = diff_grid(u1 - u0, (uint32_t)group, (uint32_t)blocks);
#define CRUM_DIFF(NTV, GV)                                                                   \
    hipLaunchKernelGGL((k_diff<NTV, GV>), dim3(nb), dim3(256), 0, s, regs, n_regs,           \
                       u0, u1, unit_flags, (uint32_t)prio, cand, stamp)
    if (nontemporal) {
        if (group == 4)
            CRUM_DIFF(true, 4);
        else if (group == 2)
            CRUM_DIFF(true, 2);
        else
            CRUM_DIFF(true, 1);
    } else {
        if (group == 4)
            CRUM_DIFF(false, 4);
        else if (group == 2)
            CRUM_DIFF(false, 2);
        else
            CRUM_DIFF(false, 1);
    }
#undef CRUM_DIFF
    return hipGetLastError();
}

// ------------------------------------------------------------ k_bitmap

// OR of the n = 2^n_shift flag bytes at f: 16 or 4 bytes at a time where they
// are aligned (a page's flags start at a multiple of n, unless smaller pages
// of another request of a plan come before it).
__device__ __forceinline__ bool any_flag(const uint8_t* __restrict__ f, uint32_t n_shift)
{
    const uint32_t n = 1u << n_shift;
    uint32_t acc = 0;
    if (n >= 16 && ((uintptr_t)f & 15u) == 0) {
        const gcv4 v = (gcv4)f;
        u32x4 o = v[0];
#pragma unroll 8
        for (uint32_t i = 1; i < n / 16; ++i)
            o |= v[i];
        acc = o.x | o.y | o.z | o.w;
    } else if (n >= 4 && ((uintptr_t)f & 3u) == 0) {
        const gcu32 v = (gcu32)f;
        for (uint32_t i = 0; i < n / 4; ++i)
            acc |= v[i];
    } else {
        for (uint32_t i = 0; i < n; ++i)
            acc |= f[i];
    }
    return acc != 0;
}

// Whether global page g exists in region R and is dirty: without a shadow every
// page is (and no flag is looked at).
__device__ __forceinline__ bool page_dirty(const DevRegion& R, uint64_t g,
                                           const uint8_t* __restrict__ unit_flags)
{
    if (g < R.first_page || g - R.first_page >= (R.len >> R.page_shift))
        return false;
    const uint32_t upp_shift = R.page_shift - R.unit_shift;
    return R.shadow == nullptr ||
           any_flag(unit_flags + R.first_unit + ((g - R.first_page) << upp_shift), upp_shift);
}

// One wave per bitmap word in [w0, w1): lane l owns global page 64w + l, and a
// ballot forms the word.  Bound by latency; 2 MiB pages (128 flags each) took
// 14-18 us a byte at a time and take 5.  (Bits set by the diff itself with atomics
// cost about 3 ns for each dirty unit: 58 us more for 8 GiB of 64 KiB pages, 9 % of them
// dirty.)
__global__ __launch_bounds__(256) void k_bitmap(const DevRegion* __restrict__ regs,
                                                uint32_t n_regs, uint64_t w0, uint64_t w1,
                                                const uint8_t* __restrict__ unit_flags,
                                                uint64_t* __restrict__ bitmap)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t w =
        w0 + (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= w1)
        return;
    const uint64_t g = w * 64 + lane;
    const uint64_t m =
        __ballot(page_dirty(regs[find_region<3>(regs, n_regs, g)], g, unit_flags));
    if (lane == 0)
        bitmap[w] = m;
}

// ------------------------------------------------------------ k_scan

// A range of at most this many bitmap words gets its slot list from k_scan
// itself (the k_list work, from LDS, with no second launch).  One workgroup
// writes the list at about 5 ns a word, so past this a separate k_list (about
// 5 us plus a launch gap) is faster.
constexpr uint64_t kScanListWords = 512;

// A range of at most this many words gets its bitmap from the unit flags in
// k_scan itself: 16 waves with 8 words each in flight, one round of three
// dependent reads, against a k_bitmap launch of 4.6 us.  A second round would cost
// as much as the launch, and so would a search over more regions than a wave
// has lanes to hold their starts.
constexpr uint64_t kScanFlagWords = 128;
constexpr uint32_t kScanFlagRegions = 64;

__global__ __launch_bounds__(1024) void k_scan(uint64_t* __restrict__ bitmap, uint64_t w0,
                                               uint64_t w1,
                                               uint32_t* __restrict__ prefix,
                                               uint64_t* __restrict__ bounds_out, int final,
                                               const DevRequest* __restrict__ reqs, uint32_t q0,
                                               uint32_t q1, DevReqOut* __restrict__ out,
                                               DevGlobal* __restrict__ glob, uint64_t capacity,
                                               int restore_mode, uint32_t* __restrict__ list,
                                               HostNote note, FlagSource fs)
{
    constexpr int V = 4;  // words per thread per pass
    static_assert(kScanListWords <= 1024 * V, "a fused list range takes one pass");
    __shared__ uint32_t wave_tot[16];
    __shared__ uint64_t s_words[kScanListWords];  // with `list`: the words and their
    __shared__ uint32_t s_pre[kScanListWords];    // prefixes, for the list below
    __shared__ uint64_t s_tot[16];
    __shared__ uint64_t s_used;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    // what the end needs, read before the words (single: one request whose last
    // word is the range's, as in every call but a plan's)
    const DevRequest& Q0 = reqs[q0];
    const bool single = final && q1 == q0 + 1 && Q0.first_word + Q0.n_words == w1;
    const uint32_t carry0 = (uint32_t)glob->running;
    const uint64_t img_next = glob->img_next, staged = glob->staging_used;
    const bool full = glob->code != 0;
    uint64_t p_first = carry0;
    if (single && Q0.first_word != w0)
        p_first = prefix[Q0.first_word];  // written by an earlier launch
    if (fs.regs) {
        const uint64_t first = lane < fs.n_regs ? fs.regs[lane].first_page : ~0ull;
        uint32_t r[kScanFlagWords / 16] = {};
        // a lane per region: the region of a word's first page by one ballot, then
        // only the regions that start inside the word are looked at one by one
        // (comparing every page with every start took 11 us for 64 regions)
#pragma unroll
        for (uint32_t i = 0; i < kScanFlagWords / 16; ++i) {
            const uint64_t p0 = (w0 + wv + 16 * i) * 64;
            if (p0 >= w1 * 64)
                break;
            r[i] = (uint32_t)__popcll(__ballot(first <= p0)) - 1;
            for (uint64_t in = __ballot(first > p0 && first <= p0 + 63); in; in &= in - 1) {
                const int k = __builtin_ctzll(in);
                const uint64_t f =
                    (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)first, k) |
                    (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(first >> 32), k)
                        << 32;
                r[i] += f <= p0 + lane;
            }
        }
#pragma unroll
        for (uint32_t i = 0; i < kScanFlagWords / 16; ++i) {
            const uint64_t w = w0 + wv + 16 * i;
            if (w < w1) {
                const uint64_t m =
                    __ballot(page_dirty(fs.regs[r[i]], w * 64 + lane, fs.unit_flags));
                if (lane == 0) {
                    bitmap[w] = m;
                    s_words[w - w0] = m;
                }
            }
        }
        __syncthreads();
    }
    uint32_t carry = carry0;
    for (uint64_t base = w0; base < w1; base += 1024 * V) {
        uint32_t c[V];
        uint32_t local = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint64_t w = base + (uint64_t)tid * V + v;
            const uint64_t word = w >= w1 ? 0ull : fs.regs ? s_words[w - w0] : bitmap[w];
            if (list && w < w1)
                s_words[w - w0] = word;
            c[v] = (uint32_t)__popcll(word);
            local += c[v];
        }
        uint32_t incl = local;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)incl, d);
            if (lane >= (uint32_t)d)
                incl += y;
        }
        if (lane == 63)
            wave_tot[wv] = incl;
        __syncthreads();
        uint32_t woff = 0, blk = 0;
        for (uint32_t i = 0; i < 16; ++i) {
            if (i < wv)
                woff += wave_tot[i];
            blk += wave_tot[i];
        }
        uint32_t excl = carry + woff + incl - local;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint64_t w = base + (uint64_t)tid * V + v;
            if (w < w1) {
                prefix[w] = excl;
                if (list)
                    s_pre[w - w0] = excl;
            }
            excl += c[v];
        }
        carry += blk;
        __syncthreads();
    }
    if (list) {
        // the k_list step: wave wv takes words 4wv .. 4wv + 3, then 64 further
        // on, ... (four LDS reads in flight); the lane of each set bit writes
        // its page at the word's prefix plus the set bits below it
        const uint64_t n = w1 - w0;
        for (uint64_t i0 = 4 * wv; i0 < n; i0 += 64) {
            uint64_t m[4];
            uint32_t pre[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                m[u] = i0 + u < n ? s_words[i0 + u] : 0ull;
                pre[u] = i0 + u < n ? s_pre[i0 + u] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(m[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[u], 0u));
                if ((m[u] >> lane) & 1u)
                    list[pre[u] + below] = (uint32_t)((w0 + i0 + u) * 64 + lane);
            }
        }
    }
    if (final && !single) {
        __threadfence_block();
        __syncthreads();
        // results of requests [q0, q1), a thread each; their images follow
        // glob->img_next, 4 KiB aligned, so an image starts at the sum of the
        // rounded sizes before it
        uint64_t img0 = img_next;
        if (tid == 0)
            s_used = staged;
        for (uint32_t base = q0; base < q1; base += 1024) {
            const uint32_t q = base + tid;
            uint64_t D = 0, p0 = 0, ib = 0, pages = 0;
            if (q < q1) {
                const DevRequest& Q = reqs[q];
                // every word of these requests lies in [.., w1): a prefix at or past
                // w1 is the running total, not a (not yet scanned) later word
                const uint64_t a = Q.first_word, b = Q.first_word + Q.n_words;
                p0 = a < w1 ? prefix[a] : carry;
                D = (b < w1 ? prefix[b] : carry) - p0;
                pages = Q.n_pages;
                ib = Q.data_off + (D << Q.page_shift) + ((4 * D + 7) & ~7ull);
            }
            const uint64_t room = (ib + 4095) & ~4095ull;
            uint64_t incl = room;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint64_t y = (uint64_t)__shfl_up((unsigned long long)incl, d);
                if (lane >= (uint32_t)d)
                    incl += y;
            }
            __syncthreads();
            if (lane == 63)
                s_tot[wv] = incl;
            __syncthreads();
            uint64_t img = img0 + incl - room;
            for (uint32_t i = 0; i < 16; ++i) {
                if (i < wv)
                    img += s_tot[i];
                img0 += s_tot[i];
            }
            if (q < q1) {
                DevReqOut& O = out[q];
                O.n_dirty = D;
                O.total_pages = pages;
                O.slot_base = p0;
                O.acc[0] = O.acc[1] = O.acc[2] = O.acc[3] = 0;
                if (!restore_mode) {
                    O.code = 0;
                    O.first_bad = 0;
                    O.image_bytes = ib;
                    O.img_base = img;
                    if (q + 1 == q1)
                        s_used = img + ib;
                }
            }
        }
        __syncthreads();
        if (!restore_mode) {
            const uint64_t used = s_used;
            if (full || used > capacity) {
                // the group does not fit: no request of it (or of a later group) is packed
                for (uint32_t q = q0 + tid; q < q1; q += 1024)
                    out[q].code = -2;  // CRUM_ENOSPC
                if (tid == 0)
                    glob->code = -2;
            } else if (tid == 0) {
                glob->staging_used = used;
                glob->img_next = img0;
            }
        }
        __threadfence_block();
        __syncthreads();
    }
    if (tid != 0)
        return;
    glob->running = carry;
    if (final)
        glob->total_dirty = carry;
    if (bounds_out)
        *bounds_out = carry;
    bool no_space = false;
    if (single) {
        DevReqOut o = out[q0];  // a restore's sizes and place are there already
        o.n_dirty = carry - p_first;
        o.total_pages = Q0.n_pages;
        o.slot_base = p_first;
        o.acc[0] = o.acc[1] = o.acc[2] = o.acc[3] = 0;
        if (!restore_mode) {
            o.first_bad = 0;
            o.image_bytes =
                Q0.data_off + (o.n_dirty << Q0.page_shift) + ((4 * o.n_dirty + 7) & ~7ull);
            o.img_base = img_next;
            const uint64_t used = img_next + o.image_bytes;
            o.code = full || used > capacity ? -2 : 0;  // CRUM_ENOSPC: nothing is packed
            if (o.code == 0) {
                glob->staging_used = used;
                glob->img_next = (used + 4095) & ~4095ull;
            } else {
                glob->code = -2;
            }
            if (note.used)
                __hip_atomic_store(note.used, o.code == 0 ? used : staged, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
        }
        out[q0] = o;
        no_space = o.code != 0 && !restore_mode;
    } else if (note.used) {
        __hip_atomic_store(note.used, glob->staging_used, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // one relaxed word: a release would write the L2 back first
    if (note.count)
        __hip_atomic_store(note.count, carry | (no_space ? kCountNoSpace : 0ull),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_scan(uint64_t* bitmap, uint64_t w0, uint64_t w1, uint32_t* prefix,
                       uint64_t* bounds_out, int final, const DevRequest* reqs, uint32_t q0,
                       uint32_t q1, DevReqOut* out, DevGlobal* glob, uint64_t capacity,
                       int restore_mode, uint32_t* list, hipStream_t s, const FlagSource& fs,
                       const HostNote& note)
{
    FlagSource in = fs;
    if (fs.regs && w1 > w0 && (w1 - w0 > kScanFlagWords || fs.n_regs > kScanFlagRegions)) {
        hipLaunchKernelGGL(k_bitmap, dim3((unsigned)((w1 - w0 + 3) / 4)), dim3(256), 0, s,
                           fs.regs, fs.n_regs, w0, w1, fs.unit_flags, bitmap);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        in.regs = nullptr;
    }
    const bool fused = list && w1 - w0 <= kScanListWords;
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, bitmap, w0, w1, prefix, bounds_out,
                       final, reqs, q0, q1, out, glob, capacity, restore_mode,
                       fused ? list : nullptr, note, in);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && list && !fused)
        e = launch_list(bitmap, prefix, w0, w1, list, s);
    return e;
}

// ------------------------------------------------------------ k_list

// Ballot compaction: the lane of each set bit writes its page index at the
// word's prefix plus the number of set bits below the lane.
__global__ __launch_bounds__(256) void k_list(const uint64_t* __restrict__ bitmap,
                                              const uint32_t* __restrict__ prefix, uint64_t w0,
                                              uint64_t w1, uint32_t* __restrict__ list)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t w =
        w0 + (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= w1)
        return;
    const uint64_t m = bitmap[w];
    if (m == 0)
        return;
    const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if ((m >> lane) & 1u)
        list[prefix[w] + below] = (uint32_t)(w * 64 + lane);
}

hipError_t launch_list(const uint64_t* bitmap, const uint32_t* prefix, uint64_t w0, uint64_t w1,
                       uint32_t* list, hipStream_t s)
{
    if (w1 <= w0)
        return hipSuccess;
    hipLaunchKernelGGL(k_list, dim3((unsigned)((w1 - w0 + 3) / 4)), dim3(256), 0, s, bitmap,
                       prefix, w0, w1, list);
    return hipGetLastError();
}

// ------------------------------------------------------------ k_pack / verify

__device__ __forceinline__ void slot_range(const SlotRange& sr, uint64_t* lo, uint64_t* hi)
{
    if (sr.bounds) {
        *lo = sr.chunk ? sr.bounds[sr.chunk - 1] : 0;
        *hi = sr.bounds[sr.chunk];
    } else {
        *lo = sr.lo;
        *hi = sr.hi;
    }
}

// A work item of k_pack found to be a piece of a page: where its bytes are and
// where they go (wave-uniform).
struct Piece {
    const uint8_t* src;   // current bytes (pack) or the packed page
    uint8_t* shadow;      // the piece's shadow, null if the region has none
    uint8_t* dst;         // its place in the image (pack) or in the region (scatter)
    uint64_t unit;        // first diff unit of the piece
    uint32_t unit_shift;
    uint32_t batches;     // 4 KiB batches in the piece
    uint32_t update;      // the shadow receives the piece's dirty units
    uint32_t region;
    uint64_t item, slot;
};

// Flag of diff unit u, read as part of an aligned word so that a wave-uniform
// u is a scalar load (a byte load counts against the vector loads in flight).
// The flags are padded to whole words.
__device__ __forceinline__ bool unit_dirty(const uint8_t* __restrict__ flags, uint64_t u)
{
    const uint32_t w = reinterpret_cast<const uint32_t*>(flags)[u >> 2];
    return (w >> (8 * (uint32_t)(u & 3))) & 0xFFu;
}

// The slot at index i of the runs laid end to end, and where its run ends.
struct RunSlot {
    uint64_t slot, run_end;
};

__device__ __forceinline__ RunSlot run_slot(const RunList& runs, uint64_t i)
{
    uint32_t r = 0;
    while (r + 1 < runs.n && i >= runs.end[r])
        ++r;
    const uint64_t base = r ? runs.end[r - 1] : 0;
    return {runs.first[r] + (i - base), runs.first[r] + (runs.end[r] - base)};
}

// Final code of a restore, once its checks are done (one thread); with h_status
// (pinned), the status goes there too.
__device__ __forceinline__ void restore_finish(DevReqOut& O, const DevGlobal& G,
                                               uint64_t* h_status)
{
    int32_t code = 0;
    uint32_t bad = 0;
    if (G.fmt_bad) {
        code = -4;  // CRUM_EFORMAT
    } else if (G.crc_bad != kNoBad) {
        code = -3;  // CRUM_ECRC
        bad = G.crc_bad;
    }
    O.code = code;
    O.first_bad = bad;
    if (h_status) {
        h_status[0] = (uint32_t)code | (uint64_t)bad << 32;
        h_status[1] = O.n_dirty;
        h_status[2] = O.total_pages;
        h_status[3] = O.image_bytes;
    }
}

// Work item = (slot, piece); pieces per slot = 2^np_shift for the launch.
// Pack: copy the dirty page into the image's page area (and the shadow) and
// write its CRC to crc_out[slot].  Verify: recompute the CRC of a packed page
// of the image and compare with the image's CRC array.  Scatter: copy the
// packed page to its page (and, with update_shadow, its shadow), unless a check
// before found the image bad; its first thread then writes the restore's status.
//
// A wave works through its items as one stream of 4 KiB batches, whichever
// page they belong to: the loads of the next batch are in flight while the
// current one is stored and folded into its CRC.
//
// Bound by memory.  A 1 KiB step of the CRC costs a wave four matrix
// instructions and about 25 vector ones, against 20 LDS lookups in byte tables
// (or 32 and more in nibble tables) before, which kept the LDS of each compute
// unit busy for about 160 cycles per KiB: the verify of 768 MB of 4 KiB pages
// went from 236 to 129 us (3.3 to 5.9 TB/s), the pack of a 1 GiB first
// snapshot (2 MiB pages) from 428 to 418 us, of 570 MB of 4 KiB pages with
// their shadows from 412 to 402.  The matrix takes 64 registers, so a SIMD
// holds four waves; their 8 KiB each in flight cover the memory's latency.
//
// RUNS: the items are the slots of up to kMaxRuns runs instead of one range,
// read from runs.host (the host image, at the same offsets) when that is given,
// and the checks note in glob->bad_call the first call that found a bad page: a
// scatter writes the runs that end before that page, and none of a later call.
// Pull: a verify that also leaves the pages in staging, so that the scatter does
// not read the host link again.
template <int MODE, bool NT_LOAD, bool NT_STORE, bool RUNS = false>
__global__ __launch_bounds__(256, 4) void k_pack(const DevRegion* __restrict__ regs, uint32_t n_regs,
                                              const DevRequest* __restrict__ reqs,
                                              DevReqOut* __restrict__ out,
                                              const uint32_t* __restrict__ list, SlotRange sr,
                                              uint32_t np_shift, uint32_t piece_shift,
                                              const uint8_t* __restrict__ unit_flags,
                                              uint8_t* __restrict__ staging,
                                              uint32_t* __restrict__ crc_out,
                                              uint32_t* __restrict__ partials,
                                              const CrcTables* __restrict__ tabs,
                                              DevGlobal* __restrict__ glob,
                                              uint32_t update_shadow, RunList runs,
                                              uint64_t* __restrict__ h_status)
{
    constexpr bool CRC = MODE != kModeScatter;
    if (MODE == kModeScatter && !RUNS && blockIdx.x == 0 && threadIdx.x == 0)
        restore_finish(out[0], *glob, h_status);
    __shared__ __attribute__((aligned(16))) uint32_t lds[CRC ? kCrcLdsWords : 4];
    if (MODE != kModePack && glob->fmt_bad)
        return;
    uint64_t slot0 = 0, slot1 = 0;
    uint64_t stop = ~0ull;  // first slot that is not written any more (scatter)
    if (RUNS) {
        slot1 = runs.end[runs.n - 1];
        if (MODE == kModeScatter && glob->crc_bad != kNoBad) {
            if (glob->bad_call < runs.call)
                return;
            stop = glob->crc_bad;
        }
    } else {
        slot_range(sr, &slot0, &slot1);
        if (MODE == kModeScatter && glob->crc_bad != kNoBad)
            return;
    }
    const uint64_t n_items = (slot1 - slot0) << np_shift;
    // a grid sized for the most slots the launch could get: workgroups past
    // the items leave before staging their tables
    if ((uint64_t)blockIdx.x * 4 >= n_items)
        return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t half = lane >> 5;
    CrcMatrix mat;
    if (CRC) {
        load_crc_matrix(mat, tabs, lane);
        load_crc_tables(lds, tabs);
    }
    const uint64_t wave =
        (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t n_waves = (uint64_t)gridDim.x * 4;
    uint32_t r = 0;
    uint64_t r_lo = 1, r_hi = 0;

    // the first item at or after `item` (this wave's items) that is a piece
    auto find = [&](uint64_t item, Piece& p) __attribute__((always_inline)) -> bool {
        for (; item < n_items; item += n_waves) {
            uint64_t k = MODE == kModeScatter && !RUNS && sr.backward
                             ? slot1 - 1 - (item >> np_shift)
                             : slot0 + (item >> np_shift);
            if (RUNS) {
                const RunSlot s = run_slot(runs, k);
                k = s.slot;
                if (MODE == kModeScatter && s.run_end > stop)
                    continue;
            }
            const uint32_t piece = (uint32_t)(item & ((1ull << np_shift) - 1));
            const uint64_t g = list[k];
            if (g < r_lo || g >= r_hi) {
                r = find_region<3>(regs, n_regs, g);
                r_lo = regs[r].first_page;
                r_hi = r_lo + (regs[r].len >> regs[r].page_shift);
            }
            const DevRegion& R = regs[r];
            if (g < r_lo || g >= r_hi)
                continue;  // only reachable for a corrupt restore bitmap (gated above)
            const DevReqOut& O = out[R.req];
            if (MODE == kModePack && O.code != 0)
                continue;  // the request's image did not fit: nothing is written
            const uint32_t ps = R.page_shift;
            const uint32_t pb_shift = ps < piece_shift ? ps : piece_shift;
            if (piece >= (1u << (ps - pb_shift)))
                continue;
            const uint64_t off = ((g - R.first_page) << ps) + ((uint64_t)piece << pb_shift);
            uint8_t* packed = staging + O.img_base + reqs[R.req].data_off +
                              ((k - O.slot_base) << ps) + ((uint64_t)piece << pb_shift);
            p.item = item;
            p.slot = k;
            p.region = r;
            p.batches = 1u << (pb_shift - 12);
            p.src = RUNS && runs.host ? runs.host + (packed - staging) : packed;
            p.dst = MODE == kModePull ? packed : nullptr;
            p.shadow = nullptr;
            p.update = 0;
            p.unit = 0;
            p.unit_shift = 0;
            if (MODE == kModeScatter) {
                p.dst = const_cast<uint8_t*>(R.cur) + off;
                p.shadow = R.shadow ? R.shadow + off : nullptr;
                p.update = update_shadow;
            }
            if (MODE == kModePack) {
                p.src = R.cur + off;
                p.dst = packed;
                p.shadow = R.shadow ? R.shadow + off : nullptr;
                p.update = R.flags & 1u;
                p.unit_shift = R.unit_shift;
                p.unit = R.first_unit + (off >> R.unit_shift);
            }
            return true;
        }
        return false;
    };
    // whether batch b of the piece lies in a diff unit that differs from the
    // shadow; a clean unit's bytes equal the shadow's
    auto dirty = [&](const Piece& p, uint32_t b) -> bool {
        return !(unit_flags && p.shadow) || unit_dirty(unit_flags, p.unit + ((b << 12) >> p.unit_shift));
    };
    // clean batches are read from the shadow, which keeps re-reads off the
    // host link when the current bytes live in host memory
    auto load = [&](const Piece& p, uint32_t b, bool d, u32x4* w) {
        const gcv4 a = (gcv4)((MODE == kModePack && !d ? p.shadow : p.src) + (b << 12)) + lane;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            w[t] = NT_LOAD ? __builtin_nontemporal_load(a + 64 * t) : a[64 * t];
    };

    auto store = [&](gv4 o, const u32x4* w) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (NT_STORE)
                __builtin_nontemporal_store(w[t], o + 64 * t);
            else
                o[64 * t] = w[t];
        }
    };

    Piece cur;
    if (!find(wave, cur))
        return;
    uint32_t b = 0, s = 0;
    bool d = MODE == kModePack ? dirty(cur, 0) : true;
    u32x4 wa[4], wb[4];
    load(cur, 0, d, wa);
    // one batch: issue the next one's loads into nx, then finish w
    auto step = [&](u32x4* w, u32x4* nx) __attribute__((always_inline)) -> bool {
        Piece next = cur;
        uint32_t nb = b + 1;
        bool more = true, nd = true;
        if (nb == cur.batches) {
            nb = 0;
            more = find(cur.item + n_waves, next);
        }
        if (more) {
            nd = MODE == kModePack ? dirty(next, nb) : true;
            load(next, nb, nd, nx);
        }
        if (MODE != kModeVerify) {
            store((gv4)(cur.dst + (b << 12)) + lane, w);
            if (cur.update && cur.shadow && d)
                store((gv4)(cur.shadow + (b << 12)) + lane, w);
        }
        if (CRC) {
            const uint32_t f = fold_4k(mat, w, half);
            s = b ? shift_4k(lds, s) ^ f : f;
        }
        if (CRC && b + 1 == cur.batches) {
            const uint32_t raw = columns_crc(lds, s, lane);
            const DevRegion& R = regs[cur.region];
            const uint32_t ps = R.page_shift;
            if (ps > piece_shift) {
                if (lane == 0)
                    partials[cur.item] = raw;
            } else {
                const DevRequest& Q = reqs[R.req];
                const uint32_t crc = raw ^ Q.init_fix;
                if (MODE == kModePack) {
                    if (lane == 0)
                        crc_out[cur.slot] = crc;
                } else {
                    const DevReqOut& O = out[R.req];
                    const uint64_t local = cur.slot - O.slot_base;
                    const uint32_t* img_crc = reinterpret_cast<const uint32_t*>(
                        staging + O.img_base + Q.data_off + (O.n_dirty << ps));
                    if (crc != img_crc[local] && lane == 0) {
                        atomicMin(&glob->crc_bad, (uint32_t)local);
                        if (RUNS)
                            atomicMin(&glob->bad_call, runs.call);
                    }
                }
            }
        }
        cur = next;
        b = nb;
        d = nd;
        return more;
    };
    while (step(wa, wb) && step(wb, wa)) {
    }
}

hipError_t launch_pack(int mode, const DevRegion* regs, uint32_t n_regs, const DevRequest* reqs,
                       DevReqOut* out, const uint32_t* list, SlotRange range,
                       uint32_t np_shift, uint32_t piece_shift, const uint8_t* unit_flags,
                       uint8_t* staging, uint32_t* crc_out, uint32_t* partials,
                       const CrcTables* tabs, DevGlobal* glob, int blocks, hipStream_t s,
                       int nt, int update_shadow, const RunList* runs, void* h_status)
{
    const uint64_t max_items = (runs ? runs->end[runs->n - 1] : range.max_slots) << np_shift;
    if (max_items == 0)
        return hipSuccess;
    if (piece_shift < kPieceShiftMin || piece_shift > kPieceShift)
        return hipErrorInvalidValue;
    const uint64_t need = (max_items + 3) / 4;
    const uint64_t nb = need < (uint64_t)blocks ? need : (uint64_t)blocks;
    const dim3 grid((unsigned)nb);
#define CRUM_PACK_R(M, L, S, F, ...)                                                           \
    hipLaunchKernelGGL((k_pack<M, L, S, ##__VA_ARGS__>), grid, dim3(256), 0, s, regs, n_regs,   \
                       reqs, out, list, range, np_shift, piece_shift, F, staging, crc_out,      \
                       partials, tabs, glob, (uint32_t)update_shadow, runs ? *runs : RunList{}, \
                       static_cast<uint64_t*>(h_status))
#define CRUM_PACK(M, L, S, F) CRUM_PACK_R(M, L, S, F)
#define CRUM_PACK_NT(M, F)                                                                     \
    switch (nt & (kPackNtLoad | kPackNtStore)) {                                               \
    case 0: CRUM_PACK(M, false, false, F); break;                                              \
    case kPackNtStore: CRUM_PACK(M, false, true, F); break;                                    \
    case kPackNtLoad: CRUM_PACK(M, true, false, F); break;                                     \
    default: CRUM_PACK(M, true, true, F); break;                                               \
    }
    if (runs) {
        if (mode == kModePull)
            CRUM_PACK_R(kModePull, false, false, nullptr, true);
        else if (mode == kModeVerify)
            CRUM_PACK_R(kModeVerify, false, false, nullptr, true);
        else
            CRUM_PACK_R(kModeScatter, false, false, nullptr, true);
    } else if (mode == kModeScatter) {
        CRUM_PACK_NT(kModeScatter, nullptr);
    } else if (mode == kModeVerify) {
        if (nt & kPackNtLoad)
            CRUM_PACK(kModeVerify, true, false, nullptr);
        else
            CRUM_PACK(kModeVerify, false, false, nullptr);
    } else {
        CRUM_PACK_NT(kModePack, unit_flags);
    }
#undef CRUM_PACK_NT
#undef CRUM_PACK_R
#undef CRUM_PACK
    return hipGetLastError();
}

// Combines the piece CRCs of the pages larger than one piece; partials are
// indexed by the item of the matching pack launch.  L = min(64, 2^np_shift)
// lanes per slot: lane l folds the pieces l, l + 64, ... (Horner, a shift by 64
// pieces per step), then pairs of neighbours, of pairs, ... combine by
// crc(A||B) = crc(A) x^(8|B|) + crc(B).  A chain of dependent products, so it
// is bound by latency: one thread per slot took 30 us for pages of 128 pieces,
// this takes 5.
template <int MODE>
__global__ __launch_bounds__(256) void k_finalize(const DevRegion* __restrict__ regs,
                                                  uint32_t n_regs,
                                                  const DevRequest* __restrict__ reqs,
                                                  const DevReqOut* __restrict__ out,
                                                  const uint32_t* __restrict__ list,
                                                  SlotRange sr, uint32_t np_shift,
                                                  uint32_t piece_shift,
                                                  const uint32_t* __restrict__ partials,
                                                  uint32_t* __restrict__ crc_out,
                                                  uint8_t* __restrict__ staging,
                                                  DevGlobal* __restrict__ glob,
                                                  const CrcTables* __restrict__ tabs,
                                                  RunList runs)
{
    if (MODE == kModeVerify && glob->fmt_bad)
        return;
    uint64_t slot0 = 0, slot1 = 0;
    if (runs.n)
        slot1 = runs.end[runs.n - 1];
    else
        slot_range(sr, &slot0, &slot1);
    const uint32_t l_shift = np_shift < 6 ? np_shift : 6;
    const uint64_t i = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> l_shift;
    const uint32_t l = threadIdx.x & ((1u << l_shift) - 1);
    // a slot's lanes stay together through the shuffles: none leaves early
    uint64_t k = slot0 + i;
    uint32_t e = 0;  // log2 of the slot's pieces, 0: nothing to combine
    uint32_t r = 0;
    if (i < slot1 - slot0) {
        if (runs.n)
            k = run_slot(runs, i).slot;
        const uint64_t g = list[k];
        r = find_region<3>(regs, n_regs, g);
        const DevRegion& R = regs[r];
        if (g >= R.first_page && g - R.first_page < (R.len >> R.page_shift) &&
            R.page_shift > piece_shift && !(MODE == kModePack && out[R.req].code != 0))
            e = R.page_shift - piece_shift;
    }
    const uint32_t np = 1u << e;
    uint32_t s = 0;
    if (e != 0 && l < np) {
        const uint32_t* p = partials + (i << np_shift) + l;
        const uint32_t K = tabs->xp[piece_shift + 6];  // x^(8 * 64 pieces)
        s = p[0];
        for (uint32_t j = 64; j < np; j += 64)
            s = gf2_mulmod(s, K) ^ p[j];
    }
    for (uint32_t v = 0; v < l_shift; ++v) {
        const uint32_t other = (uint32_t)__shfl_xor((int)s, 1 << v);
        if (v < e) {
            const bool upper = (l >> v) & 1u;
            s = gf2_mulmod(upper ? other : s, tabs->xp[piece_shift + v]) ^ (upper ? s : other);
        }
    }
    if (e == 0 || l != 0)
        return;
    const DevRegion& R = regs[r];
    const DevRequest& Q = reqs[R.req];
    const DevReqOut& O = out[R.req];
    const uint32_t crc = s ^ Q.init_fix;
    if (MODE == kModePack) {
        crc_out[k] = crc;
    } else {
        const uint64_t local = k - O.slot_base;
        const uint32_t* img_crc = reinterpret_cast<const uint32_t*>(
            staging + O.img_base + Q.data_off + (O.n_dirty << R.page_shift));
        if (crc != img_crc[local]) {
            atomicMin(&glob->crc_bad, (uint32_t)local);
            if (runs.n)
                atomicMin(&glob->bad_call, runs.call);
        }
    }
}

hipError_t launch_finalize(int mode, const DevRegion* regs, uint32_t n_regs,
                           const DevRequest* reqs, const DevReqOut* out, const uint32_t* list,
                           SlotRange range, uint32_t np_shift, uint32_t piece_shift,
                           const uint32_t* partials, uint32_t* crc_out, uint8_t* staging,
                           DevGlobal* glob, const CrcTables* tabs, hipStream_t s,
                           const RunList* runs)
{
    const uint64_t n_slots = runs ? runs->end[runs->n - 1] : range.max_slots;
    if (n_slots == 0 || np_shift == 0)
        return hipSuccess;
    const uint32_t l_shift = np_shift < 6 ? np_shift : 6;
    const unsigned nb = (unsigned)(((n_slots << l_shift) + 255) / 256);
    const RunList rl = runs ? *runs : RunList{};
    if (mode == kModePack)
        hipLaunchKernelGGL(k_finalize<kModePack>, dim3(nb), dim3(256), 0, s, regs, n_regs, reqs,
                           out, list, range, np_shift, piece_shift, partials, crc_out, staging,
                           glob, tabs, rl);
    else
        hipLaunchKernelGGL(k_finalize<kModeVerify>, dim3(nb), dim3(256), 0, s, regs, n_regs,
                           reqs, out, list, range, np_shift, piece_shift, partials, crc_out,
                           staging, glob, tabs, rl);
    return hipGetLastError();
}

// ------------------------------------------------------------ block CRC

// x^(8 * 4096 * k) mod P: a table entry per byte of k, almost always one.
__device__ __forceinline__ uint32_t xpow_batches(uint64_t k, const CrcTables* __restrict__ tabs)
{
    uint32_t v = tabs->xb[0][k & 255u];
    for (int i = 1; i < 3; ++i) {
        const uint32_t e = (uint32_t)(k >> (8 * i)) & 255u;
        if (e)
            v = gf2_mulmod(v, tabs->xb[i][e]);
    }
    return v;
}

// x^(8n) mod P for a multiple n of 4.
__device__ __forceinline__ uint32_t xpow_words(uint64_t n, const CrcTables* __restrict__ tabs)
{
    const uint32_t r = tabs->xr[(n & 4095u) >> 2];
    return n >> 12 ? gf2_mulmod(r, xpow_batches(n >> 12, tabs)) : r;
}

// A message of n bytes cut into 4 KiB batches after left-padding it with zeros
// (which leaves a raw CRC unchanged); share i of ns, one wave's, is batches
// [j0, j1).
struct MessageShare {
    uint64_t steps, j0, j1;
    int64_t pad;  // zero bytes in front of the message
    __device__ MessageShare(uint64_t n, uint32_t i, uint32_t ns)
    {
        steps = (n + 4095) >> 12;
        pad = (int64_t)(steps * 4096 - n);
        j0 = steps * i / ns;
        j1 = steps * (i + 1) / ns;
    }
    __device__ bool empty() const { return j0 >= j1; }
    // message offset of this lane's 16 bytes of step t of batch j (negative: padding)
    __device__ int64_t at(uint64_t j, int t, uint32_t lane) const
    {
        return (int64_t)((j * 256 + 64 * t + lane) * 16) - pad;
    }
};

// This wave's share of the raw CRC of a message that starts from the all-ones
// register: the raw CRC of its batches times x^(8 * bytes after them); the
// shares XOR to the whole.  load(v) gives the 16 bytes at message offset v (words
// before the message zero); use(v, w) is called on them (a store of the words, or
// nothing).  The initial register is XORed into the first word.  Uniform over
// the wave.
template <typename Load, typename Use>
__device__ __forceinline__ uint32_t message_share(const MessageShare& sp, Load load, Use use,
                                                  const CrcMatrix& mat,
                                                  const CrcTables* __restrict__ tabs,
                                                  const uint32_t* __restrict__ lds,
                                                  uint32_t lane)
{
    if (sp.empty())
        return 0;
    uint32_t s = 0;
    for (uint64_t j = sp.j0; j < sp.j1; ++j) {
        u32x4 w[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            w[t] = load(sp.at(j, t, lane));
#pragma unroll
        for (int t = 0; t < 4; ++t)
            use(sp.at(j, t, lane), w[t]);
        if (j == 0) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (sp.at(j, t, lane) + 4 * i == 0)
                        w[t][i] ^= 0xFFFFFFFFu;
        }
        const uint32_t f = fold_4k(mat, w, lane >> 5);
        s = j > sp.j0 ? shift_4k(lds, s) ^ f : f;
    }
    const uint32_t raw = columns_crc(lds, s, lane);
    const uint64_t after = sp.steps - sp.j1;
    return after ? gf2_mulmod(raw, xpow_batches(after, tabs)) : raw;
}

// Workgroups for two messages: about two 4 KiB batches for each of their
// waves, at most max.  A header of one workgroup takes 6.0 to 6.6 us, of three (64
// MiB of 4 KiB pages), which meet in atomics, 8.0, of 50 15.4: 154 batches took no
// longer with two a wave than with one.
__host__ __device__ __forceinline__ uint32_t message_blocks(uint64_t bytes_a, uint64_t bytes_b,
                                                            uint32_t max)
{
    const uint64_t want = (((bytes_a + 4095) >> 12) + ((bytes_b + 4095) >> 12) + 7) / 8;
    return want < 1 ? 1u : want < max ? (uint32_t)want : max;
}

// Which message the wave with index i of n takes a share of, and which share:
// the waves are split by the messages' batches, at least one for each message
// that is not empty.
struct WaveRole {
    bool first;  // the first message (a), else the second
    uint32_t share, shares;
    __device__ WaveRole(uint64_t bytes_a, uint64_t bytes_b, uint32_t i, uint32_t n)
    {
        const uint64_t ba = (bytes_a + 4095) >> 12, bb = (bytes_b + 4095) >> 12;
        uint32_t na = ba == 0 ? 0u : (uint32_t)((uint64_t)n * ba / (ba + bb));
        if (ba && na == 0)
            na = 1;
        if (bb && na == n)
            na = n - 1;
        first = i < na;
        share = first ? i : i - na;
        shares = first ? na : n - na;
    }
};

// Called once by every workgroup of a request after thread 0's atomics: true in
// exactly one of them, the last to arrive, which then sees every other
// workgroup's atomics.  Only atomics meet here, so thread 0 waits for its own to be
// done (a workgroup release) before it counts itself; a device fence would
// write the L2 back first, one workgroup after the other (the 8 GiB table's header
// took 13.4 us with device fences, 12.0 without; 1.5 GiB of 4 KiB pages 17.1 and
// 15.0).  Not called when a request has one workgroup.
__device__ __forceinline__ bool last_arrival(uint32_t* count, uint32_t nb, uint32_t* s_flag)
{
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        *s_flag = atomicAdd(count, 1u) == nb - 1 ? 1u : 0u;
    }
    __syncthreads();
    const bool last = *s_flag != 0;
    __syncthreads();
    return last;
}

// acc[0..3] read at L2 (device-scope atomics) by threads 0-3 at once, into
// LDS for the workgroup.
__device__ __forceinline__ void read_accs(uint32_t* acc, uint32_t* s_vals)
{
    if (threadIdx.x < 4)
        s_vals[threadIdx.x] = atomicAdd(&acc[threadIdx.x], 0u);
    __syncthreads();
}

// ------------------------------------------------------------ k_header

// nb workgroups launched per request of [q0, q0 + gridDim.x / nb), of which
// the first message_blocks() work.  Each of their waves takes a share of the CRC
// array or of the prefix (header, region table, bitmap): it writes the words into
// the image while folding them into its share of crcs_crc or meta_crc (read from
// the sources, never back from the image, which may sit in host memory).  In the meta message the header's last two words
// (meta_crc, crcs_crc) count as zero; crcs_crc is added at the end by linearity.
// With several workgroups O.acc collects the shares and the arrivals (zero on
// entry: the final scan clears it) and the last to arrive writes the two CRC
// words.
//
// Bound by latency: a chain of dependent reads, products and, with several
// workgroups, atomics.  With byte tables (44 KiB to stage) and a butterfly over
// lanes, four powers of x and five products the 64 MiB image's header took 14.6
// us and a 1.5 GiB one's of 4 KiB pages 22; now 7 and 15.
__global__ __launch_bounds__(256) void k_header(const DevRegion* __restrict__ regs,
                                                const DevRequest* __restrict__ reqs,
                                                DevReqOut* __restrict__ out,
                                                const uint64_t* __restrict__ bitmap,
                                                const uint32_t* __restrict__ crcs,
                                                uint8_t* __restrict__ staging, uint32_t q0,
                                                uint32_t nb, uint64_t capacity,
                                                const CrcTables* __restrict__ tabs,
                                                uint64_t* __restrict__ h_status)
{
    __shared__ __attribute__((aligned(16))) uint32_t lds[kCrcLdsWords];
    __shared__ uint32_t red[8];
    __shared__ uint32_t s_word;
    __shared__ uint32_t s_hdr[16];
    __shared__ uint32_t s_acc[4];
    const uint32_t q = q0 + blockIdx.x / nb, b = blockIdx.x % nb;
    const DevRequest& Q = reqs[q];
    DevReqOut& O = out[q];
    if (h_status && blockIdx.x == 0 && threadIdx.x < 4)
        h_status[threadIdx.x] = reinterpret_cast<const uint64_t*>(&O)[threadIdx.x];
    if (O.code != 0 && O.img_base + Q.data_off > capacity)
        return;  // no room even for the prefix
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t* img = staging + O.img_base;
    const uint64_t R = Q.n_regions;
    const uint64_t table_end = 64 + 32 * R;
    const uint64_t prefix_end = table_end + 8 * Q.n_words;
    const uint64_t D = O.n_dirty;
    const uint64_t first_page0 = Q.first_word * 64;
    const bool ok = O.code == 0;
    const uint64_t crc_bytes = ok ? 4 * D : 0;
    const uint32_t ne = message_blocks(crc_bytes, prefix_end, nb);
    if (b >= ne)
        return;
    const WaveRole role(crc_bytes, prefix_end, 4 * b + wave, 4 * ne);
    const MessageShare sp(role.first ? crc_bytes : prefix_end, role.share, role.shares);
    CrcMatrix mat;
    if (!sp.empty())
        load_crc_matrix(mat, tabs, lane);
    if (tid == 0) {
        s_hdr[0] = 0x4D555243u;  // "CRUM"
        s_hdr[1] = 0x31474D49u;  // "IMG1"
        s_hdr[2] = 1;
        s_hdr[3] = 1u << Q.page_shift;
        s_hdr[4] = (uint32_t)R;
        s_hdr[5] = (Q.flags & kReqShadow) ? 0u : 1u;
        s_hdr[6] = (uint32_t)Q.n_pages;
        s_hdr[7] = (uint32_t)(Q.n_pages >> 32);
        s_hdr[8] = (uint32_t)D;
        s_hdr[9] = (uint32_t)(D >> 32);
        s_hdr[10] = (uint32_t)Q.seq;
        s_hdr[11] = (uint32_t)(Q.seq >> 32);
        s_hdr[12] = (uint32_t)Q.data_off;
        s_hdr[13] = (uint32_t)(Q.data_off >> 32);
        s_hdr[14] = 0;
        s_hdr[15] = 0;
    }
    load_crc_tables(lds, tabs);

    uint32_t share = 0;
    if (role.first) {
        uint8_t* dst = img + Q.data_off + (D << Q.page_shift);
        const gcu32 src = (gcu32)(crcs + O.slot_base);
        const bool even = (D & 1) == 0;  // then the pad, and every v, is a multiple of 8
        auto load = [&](int64_t v) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w[i] = v + 4 * i >= 0 ? src[(v >> 2) + i] : 0u;
            return w;
        };
        auto use = [&](int64_t v, u32x4 w) {
            if (even) {
                if (v >= 0)
                    *(gv2)(dst + v) = u32x2{w.x, w.y};
                if (v + 8 >= 0)
                    *(gv2)(dst + v + 8) = u32x2{w.z, w.w};
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (v + 4 * i >= 0)
                        ((gu32)dst)[(v >> 2) + i] = w[i];
            }
        };
        share = message_share(sp, load, use, mat, tabs, lds, lane);
        if (role.share == 0 && lane == 0 && !even)
            ((gu32)dst)[D] = 0;
    } else {
        // prefix word at byte r: header, region table entries {id, len, first
        // page within the request, 0}, then the bitmap
        const gcu32 bm32 = (gcu32)(bitmap + Q.first_word);
        auto prefix_word = [&](uint64_t r) -> uint32_t {
            if (r >= table_end)
                return bm32[(r - table_end) >> 2];
            if (r < 64)
                return s_hdr[r >> 2];
            const uint64_t t = r - 64;
            const DevRegion& G = regs[Q.first_region + (t >> 5)];
            const uint32_t k = (uint32_t)(t >> 2) & 7u;
            const uint64_t v =
                k < 2 ? G.id : k < 4 ? G.len : k < 6 ? G.first_page - first_page0 : 0;
            return (uint32_t)(v >> (32 * (k & 1)));
        };
        // the prefix is a multiple of 8 bytes, so each lane's 16 are two aligned
        // 8-byte pairs; the pair at 56 is the two CRC words, written last
        auto load = [&](int64_t v) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w[i] = v + 4 * i >= 0 ? prefix_word((uint64_t)(v + 4 * i)) : 0u;
            return w;
        };
        auto use = [&](int64_t v, u32x4 w) {
            if (v >= 0 && v != 56)
                *(gv2)(img + v) = u32x2{w.x, w.y};
            if (v + 8 >= 0 && v + 8 != 56)
                *(gv2)(img + v + 8) = u32x2{w.z, w.w};
        };
        share = message_share(sp, load, use, mat, tabs, lds, lane);
    }
    if (lane == 0) {
        red[wave] = role.first ? share : 0;
        red[4 + wave] = role.first ? 0 : share;
    }
    const uint64_t gt = (uint64_t)b * blockDim.x + tid, gstride = (uint64_t)ne * blockDim.x;
    for (uint64_t o = prefix_end + 8 * gt; o < Q.data_off; o += 8 * gstride)
        *reinterpret_cast<uint64_t*>(img + o) = 0;
    __syncthreads();
    uint32_t c_raw = red[0] ^ red[1] ^ red[2] ^ red[3];
    uint32_t m_raw = red[4] ^ red[5] ^ red[6] ^ red[7];
    if (ne > 1) {
        if (tid == 0) {
            if (c_raw)
                atomicXor(&O.acc[0], c_raw);
            if (m_raw)
                atomicXor(&O.acc[1], m_raw);
        }
        if (!last_arrival(&O.acc[2], ne, &s_word))
            return;
        read_accs(O.acc, s_acc);
        c_raw = s_acc[0];
        m_raw = s_acc[1];
    }
    if (tid == 0) {
        const uint32_t crcs_crc = crc_bytes ? c_raw ^ 0xFFFFFFFFu : 0u;
        const uint32_t meta =
            m_raw ^ gf2_mulmod(crcs_crc, xpow_words(prefix_end - 60, tabs)) ^ 0xFFFFFFFFu;
        *(gv2)(img + 56) = u32x2{meta, crcs_crc};
    }
}

// Workgroups per request for the header and image-check kernels.
uint32_t header_blocks(uint64_t n_regions, uint64_t n_words, uint64_t n_crcs)
{
    return message_blocks(4 * n_crcs, 64 + 32 * n_regions + 8 * n_words, 128);
}

hipError_t launch_header(const DevRegion* regs, const DevRequest* reqs, uint32_t q0, uint32_t q1,
                         uint32_t blocks, DevReqOut* out, const uint64_t* bitmap,
                         const uint32_t* crcs, uint8_t* staging, uint64_t capacity,
                         const CrcTables* tabs, hipStream_t s, void* h_status)
{
    if (q1 <= q0)
        return hipSuccess;
    if (blocks == 0 || (uint64_t)(q1 - q0) * blocks > 0x7FFFFFFFull)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_header, dim3((q1 - q0) * blocks), dim3(256), 0, s, regs, reqs, out,
                       bitmap, crcs, staging, q0, blocks, capacity, tabs,
                       static_cast<uint64_t*>(h_status));
    return hipGetLastError();
}

__global__ void k_plan_init(DevGlobal* __restrict__ glob)
{
    glob->total_dirty = 0;
    glob->staging_used = 0;
    glob->code = 0;
    glob->fmt_bad = 0;
    glob->crc_bad = kNoBad;
    glob->running = 0;
    glob->img_next = 0;
}

hipError_t launch_plan_init(DevGlobal* glob, hipStream_t s)
{
    hipLaunchKernelGGL(k_plan_init, dim3(1), dim3(1), 0, s, glob);
    return hipGetLastError();
}

__global__ void k_plan_status(const DevReqOut* __restrict__ out, uint32_t n,
                              uint8_t* __restrict__ dst)
{
    const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n)
        return;
    const DevReqOut& O = out[q];
    uint8_t* d = dst + 40ull * q;
    *reinterpret_cast<int32_t*>(d) = O.code;
    *reinterpret_cast<uint32_t*>(d + 4) = O.first_bad;
    *reinterpret_cast<uint64_t*>(d + 8) = O.n_dirty;
    *reinterpret_cast<uint64_t*>(d + 16) = O.total_pages;
    *reinterpret_cast<uint64_t*>(d + 24) = O.image_bytes;
    *reinterpret_cast<uint64_t*>(d + 32) = O.img_base;
}

hipError_t launch_plan_status(const DevReqOut* out, uint32_t n, uint8_t* dst, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_plan_status, dim3((n + 255) / 256), dim3(256), 0, s, out, n, dst);
    return hipGetLastError();
}

// ------------------------------------------------------------ restore

// Device-side image checks that need the bytes: meta_crc, crcs_crc, bitmap
// population and unused bits, zero pads.  The host has already checked the
// header fields, lengths and the region table.  nb workgroups launched per
// request, of which the first message_blocks() work; each takes a share of the
// bitmap, the pad and the two CRC messages.  With several, O.acc (zero on
// entry: the host uploads it cleared) collects the CRC shares, the arrivals
// and the population, and the last workgroup to arrive compares.
__global__ __launch_bounds__(256) void k_restore_check(const DevRequest* __restrict__ reqs,
                                                       DevReqOut* __restrict__ out,
                                                       const uint8_t* __restrict__ staging,
                                                       uint32_t nb,
                                                       const CrcTables* __restrict__ tabs,
                                                       DevGlobal* __restrict__ glob)
{
    __shared__ __attribute__((aligned(16))) uint32_t lds[kCrcLdsWords];
    __shared__ uint32_t red[8];
    __shared__ uint32_t s_pop;
    __shared__ uint32_t s_word;
    __shared__ uint32_t s_acc[4];
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t q = blockIdx.x / nb, b = blockIdx.x % nb;
    const DevRequest& Q = reqs[q];
    DevReqOut& O = out[q];
    const uint8_t* img = staging + O.img_base;
    const gcu32 img32 = (gcu32)img;
    const uint64_t R = Q.n_regions;
    const uint64_t prefix_end = 64 + 32 * R + 8 * Q.n_words;
    const uint64_t D = reinterpret_cast<const uint64_t*>(img)[4];
    const uint64_t crcs_off = Q.data_off + (D << Q.page_shift);
    const uint32_t ne = message_blocks(4 * D, prefix_end, nb);
    if (b >= ne)
        return;
    const WaveRole role(4 * D, prefix_end, 4 * b + wave, 4 * ne);
    const MessageShare sp(role.first ? 4 * D : prefix_end, role.share, role.shares);
    CrcMatrix mat;
    if (!sp.empty())
        load_crc_matrix(mat, tabs, lane);
    if (tid == 0)
        s_pop = 0;
    load_crc_tables(lds, tabs);

    const uint64_t gt = (uint64_t)b * blockDim.x + tid, gstride = (uint64_t)ne * blockDim.x;
    const uint64_t* bm = reinterpret_cast<const uint64_t*>(img + 64 + 32 * R);
    uint32_t pop = 0, bad = 0;
    for (uint64_t w = gt; w < Q.n_words; w += gstride) {
        const uint64_t word = bm[w];
        pop += (uint32_t)__popcll(word);
        if (w == Q.n_words - 1 && (Q.n_pages & 63)) {
            if (word >> (Q.n_pages & 63))
                bad = 1;
        }
    }
    for (uint64_t o = prefix_end + 8 * gt; o < Q.data_off; o += 8 * gstride)
        if (*reinterpret_cast<const uint64_t*>(img + o))
            bad = 1;
    if (gt == 0) {
        for (uint64_t o = crcs_off + 4 * D; o < O.image_bytes; ++o)
            if (img[o])
                bad = 1;
    }
    if (bad)
        atomicOr(&glob->fmt_bad, 1u);
    if (pop)
        atomicAdd(&s_pop, pop);

    // the CRC array, or the prefix (where meta_crc itself reads as zero)
    const gcu32 src = role.first ? (gcu32)(img + crcs_off) : img32;
    const int64_t zero_at = role.first ? -1 : 56;
    auto load = [&](int64_t v) {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t r = v + 4 * i;
            w[i] = r >= 0 && r != zero_at ? src[r >> 2] : 0u;
        }
        return w;
    };
    const uint32_t share =
        message_share(sp, load, [](int64_t, u32x4) {}, mat, tabs, lds, lane);
    if (lane == 0) {
        red[wave] = role.first ? share : 0;
        red[4 + wave] = role.first ? 0 : share;
    }
    __syncthreads();
    uint32_t c_raw = red[0] ^ red[1] ^ red[2] ^ red[3];
    uint32_t m_raw = red[4] ^ red[5] ^ red[6] ^ red[7], total_pop = s_pop;
    if (ne > 1) {
        if (tid == 0) {
            if (c_raw)
                atomicXor(&O.acc[0], c_raw);
            if (m_raw)
                atomicXor(&O.acc[1], m_raw);
            if (s_pop)
                atomicAdd(&O.acc[3], s_pop);
        }
        if (!last_arrival(&O.acc[2], ne, &s_word))
            return;
        read_accs(O.acc, s_acc);
        c_raw = s_acc[0];
        m_raw = s_acc[1];
        total_pop = s_acc[3];
    }
    if (tid == 0) {
        const uint32_t crcs = D ? c_raw ^ 0xFFFFFFFFu : 0u;
        const uint32_t meta = m_raw ^ 0xFFFFFFFFu;
        if ((uint64_t)total_pop != D || crcs != img32[15] || meta != img32[14])
            atomicOr(&glob->fmt_bad, 1u);
    }
}

hipError_t launch_restore_check(const DevRequest* reqs, uint32_t n_reqs, uint32_t blocks,
                                DevReqOut* out, const uint8_t* staging, const CrcTables* tabs,
                                DevGlobal* glob, hipStream_t s)
{
    if (n_reqs == 0)
        return hipSuccess;
    if (blocks == 0 || (uint64_t)n_reqs * blocks > 0x7FFFFFFFull)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_restore_check, dim3(n_reqs * blocks), dim3(256), 0, s, reqs, out,
                       staging, blocks, tabs, glob);
    return hipGetLastError();
}

__global__ void k_restore_finish(DevReqOut* __restrict__ out, DevGlobal* __restrict__ glob,
                                 uint64_t* __restrict__ h_status)
{
    restore_finish(out[0], *glob, h_status);
}

hipError_t launch_restore_finish(DevReqOut* out, uint32_t, DevGlobal* glob, hipStream_t s,
                                 void* h_status)
{
    hipLaunchKernelGGL(k_restore_finish, dim3(1), dim3(1), 0, s, out, glob,
                       static_cast<uint64_t*>(h_status));
    return hipGetLastError();
}

}  // namespace crum
