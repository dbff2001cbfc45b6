// sha256_batch.hip -- SHA-256 of many independent messages, one lane each.
//
// FIPS 180-4: padding (Sec. 5.1.1), parsing into 512-bit blocks of sixteen
// big-endian words (Sec. 5.2.1), the message schedule and 64 rounds of the
// hash computation (Sec. 6.2.2) with the functions of Sec. 4.1.2.  The round
// constants (Sec. 4.2.2) and the initial hash value (Sec. 5.3.3) are derived
// at compile time from their definitions.
//
// gfx950 mapping, many messages: a lane owns one message and keeps the eight
// working variables and a rolling 16-word schedule in registers; the 64 rounds
// are unrolled so every K_t is an instruction literal.  Rotations are single
// v_alignbit_b32, Ch / Maj / three-way XORs single v_bitop3_b32, and the sums
// v_add3_u32.  The host orders a launch's messages longest first, so lanes of
// a wave run for similar lengths.  Bound by VALU issue: 1402 instructions per
// block, 512 MiB in 4 KiB messages in 369 us = 1455 GB/s of the 1795 that
// 64 lanes per clock at 2.4 GHz would give.  Few messages: bound by one
// message's chain of blocks, see sha256_split_kernel.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "shabatch_internal.h"

namespace aesctr {
namespace {

// ---- Constants from their definitions (compile time) --------------------

constexpr bool is_prime(uint32_t n)
{
    if (n < 2)
        return false;
    for (uint32_t d = 2; d * d <= n; ++d)
        if (n % d == 0)
            return false;
    return true;
}

constexpr uint32_t nth_prime(int i)
{
    uint32_t n = 1;
    for (int found = -1; found < i;)
        if (is_prime(++n))
            ++found;
    return n;
}

// floor(x^(1/e)) for e = 2, 3 by bisection over exact 128-bit integers.
constexpr uint64_t int_root(unsigned __int128 x, int e)
{
    uint64_t lo = 0, hi = uint64_t(1) << 40;
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo + 1) / 2;
        unsigned __int128 p = static_cast<unsigned __int128>(mid) * mid;
        if (e == 3)
            p *= mid;
        if (p <= x)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// First 32 bits of the fractional part of the e-th root of p.
constexpr uint32_t frac_bits(uint32_t p, int e)
{
    return static_cast<uint32_t>(int_root(static_cast<unsigned __int128>(p) << (32 * e), e));
}

struct ShaConsts {
    uint32_t k[64];
    uint32_t h0[8];
};

constexpr ShaConsts make_consts()
{
    ShaConsts c{};
    for (int i = 0; i < 64; ++i)
        c.k[i] = frac_bits(nth_prime(i), 3);
    for (int i = 0; i < 8; ++i)
        c.h0[i] = frac_bits(nth_prime(i), 2);
    return c;
}

constexpr ShaConsts kSha = make_consts();
static_assert(nth_prime(63) == 311, "the 64th prime");

// ---- Round functions -------------------------------------------------------

__device__ __forceinline__ uint32_t rotr(uint32_t x, int n) { return __builtin_amdgcn_alignbit(x, x, n); }

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Ch(x,y,z) = x ? y : z per bit; Maj = majority (bitop3 truth tables indexed
// by x<<2 | y<<1 | z).
__device__ __forceinline__ uint32_t ch(uint32_t x, uint32_t y, uint32_t z)
{
    return __builtin_amdgcn_bitop3_b32(x, y, z, 0xCA);
}

__device__ __forceinline__ uint32_t maj(uint32_t x, uint32_t y, uint32_t z)
{
    return __builtin_amdgcn_bitop3_b32(x, y, z, 0xE8);
}

__device__ __forceinline__ uint32_t bsig0(uint32_t x) { return xor3(rotr(x, 2), rotr(x, 13), rotr(x, 22)); }
__device__ __forceinline__ uint32_t bsig1(uint32_t x) { return xor3(rotr(x, 6), rotr(x, 11), rotr(x, 25)); }
__device__ __forceinline__ uint32_t ssig0(uint32_t x) { return xor3(rotr(x, 7), rotr(x, 18), x >> 3); }
__device__ __forceinline__ uint32_t ssig1(uint32_t x) { return xor3(rotr(x, 17), rotr(x, 19), x >> 10); }

__device__ __forceinline__ uint32_t add3(uint32_t a, uint32_t b, uint32_t c) { return a + b + c; }

__device__ __forceinline__ uint32_t bswap(uint32_t x) { return __builtin_amdgcn_perm(x, x, 0x00010203u); }

// W_t = s1(W_{t-2}) + W_{t-7} + s0(W_{t-15}) + W_{t-16} from the sixteen words
// before it, which roll in place.
__device__ __forceinline__ uint32_t next_word(const uint32_t w[16], int t)
{
    return add3(ssig1(w[(t - 2) & 15]), w[(t - 7) & 15], ssig0(w[(t - 15) & 15])) + w[t & 15];
}

// One of the 64 rounds (Sec. 6.2.2, step 3) on the working variables a..h =
// s[0..7], with kw = W_t + K_t.
__device__ __forceinline__ void sha_round(uint32_t s[8], uint32_t kw)
{
    const uint32_t t1 = add3(s[7], bsig1(s[4]), ch(s[4], s[5], s[6])) + kw;
    const uint32_t t2 = bsig0(s[0]) + maj(s[0], s[1], s[2]);
    s[7] = s[6];
    s[6] = s[5];
    s[5] = s[4];
    s[4] = s[3] + t1;
    s[3] = s[2];
    s[2] = s[1];
    s[1] = s[0];
    s[0] = t1 + t2;
}

// One 512-bit block: w[0..15] are the block's big-endian words.
__device__ __forceinline__ void compress(uint32_t H[8], uint32_t w[16])
{
    uint32_t s[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) s[j] = H[j];
#pragma unroll
    for (int t = 0; t < 64; ++t) {
        if (t >= 16)
            w[t & 15] = next_word(w, t);
        sha_round(s, kSha.k[t] + w[t & 15]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) H[j] += s[j];
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Messages and digests start at any byte: 4- and 16-byte accesses of byte
// alignment (gfx950 takes them at any address).  The global address space
// keeps them global_* rather than flat_*.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef const __attribute__((address_space(1))) u32x4_any g_cu32x4;
typedef __attribute__((address_space(1))) u32x4_any g_u32x4;
typedef const __attribute__((address_space(1))) u32_any g_cu32;
typedef const __attribute__((address_space(1))) uint8_t g_cu8;

__device__ __forceinline__ g_cu8 *msg_ptr(uint64_t in) { return reinterpret_cast<g_cu8 *>(static_cast<uintptr_t>(in)); }

// The sixteen words of a full block at p, as they lie in memory.  Ordinary loads: a
// lane comes back to a 128-byte line for the next block, and off alignment for a
// third one, which a non-temporal hint has read from memory again (131,072 messages
// of 4 KiB 408 us a call instead of 374, one byte off alignment 442 instead of 386).
__device__ __forceinline__ void load_raw(g_cu8 *p, u32x4 d[4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
        d[i] = reinterpret_cast<g_cu32x4 *>(p)[i];
}

__device__ __forceinline__ void to_words(const u32x4 d[4], uint32_t w[16])
{
#pragma unroll
    for (int i = 0; i < 16; ++i)
        w[i] = bswap(d[i >> 2][i & 3]);
}

// Blocks of a message once padded, and the whole blocks of data before its
// padding (Sec. 5.1.1).
__device__ __forceinline__ uint64_t padded_blocks(uint64_t len) { return (len + 8) / 64 + 1; }
__device__ __forceinline__ uint64_t data_blocks(uint64_t len) { return len >> 6; }

// The block after the last whole one: the rest (< 64 bytes, at p) of the
// message, the 0x80 byte and zeros; with the 64-bit big-endian bit length
// when it still fits.  When it does not (rest >= 56) one more block follows,
// of zeros and the length (length_block).  Whole words are read as words, the
// last one to three bytes one by one: nothing past the message is read.
__device__ __forceinline__ void tail_words(g_cu8 *p, uint64_t len, uint32_t w[16])
{
    const uint32_t rest = static_cast<uint32_t>(len & 63), part = rest >> 2;
    uint32_t v = 0x80u << (24 - 8 * (rest & 3));
#pragma unroll
    for (uint32_t j = 0; j < 3; ++j)
        if (j < (rest & 3))
            v |= uint32_t(p[4 * part + j]) << (24 - 8 * j);
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) {
        w[i] = i == part ? v : 0;
        if (i < part)
            w[i] = bswap(*reinterpret_cast<g_cu32 *>(p + 4 * i));
    }
    if (rest < 56) {
        w[14] = static_cast<uint32_t>(len >> 29);
        w[15] = static_cast<uint32_t>(len << 3);
    }
}

__device__ __forceinline__ void length_block(uint64_t len, uint32_t w[16])
{
#pragma unroll
    for (int i = 0; i < 14; ++i) w[i] = 0;
    w[14] = static_cast<uint32_t>(len >> 29);
    w[15] = static_cast<uint32_t>(len << 3);
}

// Four digest words, big-endian.
__device__ __forceinline__ void store_words(uint64_t to, const uint32_t H[4])
{
    *reinterpret_cast<g_u32x4 *>(static_cast<uintptr_t>(to)) = u32x4{bswap(H[0]), bswap(H[1]), bswap(H[2]), bswap(H[3])};
}

// One lane per message.  The next block's loads, and the tail's, are in
// flight while a block compresses; the one or two padding blocks run in a
// loop of their own, so a wave pays for them once whatever its lanes' lengths.
// Messages at any address take the same 16-byte loads (64 byte loads per block
// before: 65,536 messages of 4 KiB one byte off alignment 238 -> 206 us a call, aligned
// ones 228 -> 194).
__global__ __launch_bounds__(256) void sha256_batch_kernel(const ShaRecord *__restrict__ recs, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const ShaRecord r = recs[i];
        g_cu8 *p = msg_ptr(r.in);
        const uint64_t full = data_blocks(r.len);
        u32x4 nx[4];
        if (full > 0)
            load_raw(p, nx);
        uint32_t w[16], tail[16];
        tail_words(p + 64 * full, r.len, tail);
        uint32_t H[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) H[j] = kSha.h0[j];
        if (full > 0) {
            to_words(nx, w);
            for (uint64_t blk = 1; blk < full; ++blk) {
                load_raw(p + 64 * blk, nx);
                compress(H, w);
                to_words(nx, w);
            }
            compress(H, w);
        }
        for (uint64_t blk = full;;) {
            compress(H, tail);
            if (++blk == padded_blocks(r.len))
                break;
            length_block(r.len, tail);
        }
        store_words(r.digest, H);
        store_words(r.digest + 16, H + 4);
    }
}

// ---- Few messages: three waves per 64 messages ------------------------------

// A message's blocks are a serial chain, so with fewer messages than the chip
// has lanes the time is the longest message's blocks times one block's
// latency on one wave: about 1400 VALU instructions of four clocks.  A third
// of them, the message schedule, does not depend on the hash state, and half
// of a round does not depend on the other half.  So a workgroup of three
// waves takes 64 messages:
//  * wave 0 (lane l: message l) loads the blocks, expands their schedules and
//    writes W_t + K_t to LDS, ahead of the others;
//  * waves 1 and 2 run the 64 rounds of 32 messages each, two lanes to a
//    message: one holds a, b, c, d and computes S0(a) + Maj(a,b,c), the other
//    e, f, g, h and S1(e) + Ch(e,f,g) + h + W + K, with the same instructions
//    (rotation counts in registers); DPP moves exchange the sums.  A round is
//    11 instructions instead of 14.
// Three buffers of 16 KiB and one barrier per block: after the barrier that
// ends trip b the words of blocks b and b + 1 are complete, so the rounds of
// block b never wait for the reads of the next block's first words.
// Measured per block of the longest message: 1.48 us, against 2.85 for one
// lane per message (3.4 with byte loads); 1.70 with one lane to a message in a
// single round wave of 14 instructions per round.
constexpr int kSplitWG = 192;
constexpr int kBlockQuads = 16;    // 64 words W_t + K_t as 16-byte quads
constexpr int kAhead = 4;          // quads a round wave holds in advance

// DPP: lanes 0-3 and 8-11 of a row of 16 hold a..d (banks 0 and 2), the lanes
// four up hold e..h of the same messages.
#define SHA_FROM_E "row_shl:4 row_mask:0xf bank_mask:0x5"    // a..d lanes read their e..h lane
#define SHA_FROM_A "row_shr:4 row_mask:0xf bank_mask:0xa"    // e..h lanes read their a..d lane
#define SHA_E_ONLY "quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0xa"

// What a lane's half of the rounds needs: rotation counts, and a mask that is
// all ones on a..d lanes (Maj(x,y,z) = ~(x ^ y) ? y : z, Ch(x,y,z) = x ? y : z).
struct HalfRound {
    uint32_t n1, n2, n3, maj_mask;
};

// Eight rounds on x, y, z, w = a, b, c, d or e, f, g, h (s[0..3]); hk is
// h + W_t + K_t on e..h lanes and dd their d; both are 0 on a..d lanes, and
// come out for the round after.  kw[j]: W + K of round t + 1 + j.  One block,
// so that the order stays: a lone wave loses 1.6 clocks to an instruction that
// uses the result just before it (a chain of v_bitop3_b32 takes 5.6 clocks per
// instruction, independent ones 4.1), and a DPP source must be two
// instructions old.  The variables stay where they are and change names: a
// round's w register takes the new x.
__device__ __forceinline__ void half_rounds8(uint32_t s[4], uint32_t &hk, uint32_t &dd, const HalfRound &c,
                                             const uint32_t kw[8])
{
    uint32_t t0, t1, t2, t3, hk2 = 0, dd2 = 0;
#define SHA_HALF(x, y, z, w, hk, hk2, dd, dd2, kw)                                                        \
    "v_alignbit_b32 %[t0], %[" #x "], %[" #x "], %[n1]\n\t"                                               \
    "v_alignbit_b32 %[t1], %[" #x "], %[" #x "], %[n2]\n\t"                                               \
    "v_alignbit_b32 %[t2], %[" #x "], %[" #x "], %[n3]\n\t"                                               \
    "v_bitop3_b32 %[t3], %[" #x "], %[" #y "], %[mm] bitop3:0xd2\n\t"                                     \
    "v_bitop3_b32 %[t0], %[t0], %[t1], %[t2] bitop3:0x96\n\t"                                             \
    "v_bitop3_b32 %[t3], %[t3], %[" #y "], %[" #z "] bitop3:0xca\n\t"                                     \
    "v_add_u32_dpp %[" #hk2 "], %[" #z "], %[" #kw "] " SHA_E_ONLY "\n\t"                                 \
    "v_add3_u32 %[t0], %[t0], %[t3], %[" #hk "]\n\t"                                                      \
    "v_mov_b32_dpp %[" #dd2 "], %[" #z "] " SHA_FROM_A "\n\t"                                             \
    "v_add_u32 %[" #w "], %[t0], %[" #dd "]\n\t"                                                          \
    "v_add_u32_dpp %[" #w "], %[t0], %[" #w "] " SHA_FROM_E "\n\t"
    asm("s_nop 1\n\t"
        SHA_HALF(x, y, z, w, ha, hb, da, db, k0)
        SHA_HALF(w, x, y, z, hb, ha, db, da, k1)
        SHA_HALF(z, w, x, y, ha, hb, da, db, k2)
        SHA_HALF(y, z, w, x, hb, ha, db, da, k3)
        SHA_HALF(x, y, z, w, ha, hb, da, db, k4)
        SHA_HALF(w, x, y, z, hb, ha, db, da, k5)
        SHA_HALF(z, w, x, y, ha, hb, da, db, k6)
        SHA_HALF(y, z, w, x, hb, ha, db, da, k7)
        : [x] "+&v"(s[0]), [y] "+&v"(s[1]), [z] "+&v"(s[2]), [w] "+&v"(s[3]), [ha] "+&v"(hk), [hb] "+&v"(hk2),
          [da] "+&v"(dd), [db] "+&v"(dd2), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)
        : [n1] "v"(c.n1), [n2] "v"(c.n2), [n3] "v"(c.n3), [mm] "v"(c.maj_mask), [k0] "v"(kw[0]), [k1] "v"(kw[1]),
          [k2] "v"(kw[2]), [k3] "v"(kw[3]), [k4] "v"(kw[4]), [k5] "v"(kw[5]), [k6] "v"(kw[6]), [k7] "v"(kw[7]));
#undef SHA_HALF
}

__global__ __launch_bounds__(kSplitWG) void sha256_split_kernel(const ShaRecord *__restrict__ recs, uint32_t n)
{
    __shared__ u32x4 s_kw[3][kBlockQuads][64];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Message of this lane among the workgroup's 64, and whether a round lane
    // holds e..h.
    const uint32_t m = wave == 0 ? lane : 32 * (wave - 1) + 4 * (lane >> 3) + (lane & 3);
    const bool e_lane = (lane & 4) != 0;
    const uint32_t i = blockIdx.x * 64 + m;
    const ShaRecord r = i < n ? recs[i] : ShaRecord{0, 0, 0, 0};
    const uint64_t blocks = i < n ? padded_blocks(r.len) : 0;
    // Trips of all three waves: the longest message of the 64.
    __shared__ uint64_t s_trips;
    if (wave == 0) {
        uint64_t longest = blocks;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const uint64_t o = __shfl_xor(longest, d);
            longest = o > longest ? o : longest;
        }
        if (lane == 0)
            s_trips = longest;
    }
    __syncthreads();
    const uint64_t trips = s_trips;
    if (wave == 0) {
        g_cu8 *p = msg_ptr(r.in);
        const uint64_t full = i < n ? data_blocks(r.len) : 0;
        // Data two blocks ahead: a block's trip may be shorter than a read
        // from memory.
        u32x4 a[4] = {}, b[4] = {};
        if (full > 0)
            load_raw(p, a);
        if (full > 1)
            load_raw(p + 64, b);
        uint32_t tail[16] = {};
        if (i < n)
            tail_words(p + 64 * full, r.len, tail);
        uint32_t buf = 0;
        auto produce = [&](uint64_t blk, u32x4 (&d)[4]) {
            u32x4 (*kw)[64] = s_kw[buf];
            buf = buf == 2 ? 0 : buf + 1;
            uint32_t w[16];
            to_words(d, w);
            if (blk + 2 < full)
                load_raw(p + 64 * (blk + 2), d);
            if (blk == full) {
#pragma unroll
                for (int j = 0; j < 16; ++j) w[j] = tail[j];
            }
            if (blk > full)
                length_block(r.len, w);
#pragma unroll
            for (int q = 0; q < kBlockQuads; ++q) {
                u32x4 v;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 4 * q + j;
                    if (t >= 16)
                        w[t & 15] = next_word(w, t);
                    v[j] = w[t & 15] + kSha.k[t];
                }
                kw[q][lane] = v;
            }
            __syncthreads();
        };
        // Block 0, then block b + 1 while the other waves run block b's
        // rounds: trips + 1 barriers, as on their side.
        for (uint64_t blk = 0; blk < trips; blk += 2) {
            produce(blk, a);
            if (blk + 1 < trips)
                produce(blk + 1, b);
        }
        __syncthreads();
    } else {
        const HalfRound c = e_lane ? HalfRound{6, 11, 25, 0} : HalfRound{2, 13, 22, ~0u};
        uint32_t H[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) H[j] = e_lane ? kSha.h0[4 + j] : kSha.h0[j];
        __syncthreads();    // block 0 is there
        u32x4 first[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) first[q] = s_kw[0][q][m];
        uint32_t buf = 0;
        for (uint64_t blk = 0; blk < trips; ++blk) {
            __syncthreads();    // block blk + 1 is there (or there is none)
            const u32x4 (*kw)[64] = s_kw[buf];
            buf = buf == 2 ? 0 : buf + 1;
            u32x4 v[kBlockQuads];
#pragma unroll
            for (int q = 0; q < kBlockQuads; ++q)
                v[q] = q < kAhead ? first[q] : kw[q][m];
            uint32_t s[4] = {H[0], H[1], H[2], H[3]};
            uint32_t hk = e_lane ? s[3] + v[0][0] : 0;
            uint32_t dd = __builtin_amdgcn_update_dpp(0, s[3], 0x114, 0xf, 0xa, false);    // row_shr:4, e..h lanes
#pragma unroll
            for (int t = 0; t < 64; t += 8) {
                uint32_t next[8];    // W + K of rounds t + 1 .. t + 8
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    next[j] = t + j < 63 ? v[(t + j + 1) >> 2][(t + j + 1) & 3] : 0;
                // Past the last block the next buffer's words go unused.
                if (t == 48) {
#pragma unroll
                    for (int q = 0; q < kAhead; ++q) first[q] = s_kw[buf][q][m];
                }
                half_rounds8(s, hk, dd, c, next);
            }
            if (blk < blocks) {
#pragma unroll
                for (int j = 0; j < 4; ++j) H[j] += s[j];
            }
        }
        if (i < n)
            store_words(r.digest + (e_lane ? 16 : 0), H);
    }
}

}  // namespace

int launch_sha256_batch(const ShaRecord *dev_recs, uint32_t n, int grid, bool split, hipStream_t st)
{
    if (grid <= 0 || n == 0)
        return AES_EINVAL;
    (void)hipGetLastError();   // not ours: left by earlier calls
    if (split) {
        hipLaunchKernelGGL(sha256_split_kernel, dim3((n + 63) / 64), dim3(kSplitWG), 0, st, dev_recs, n);
        return launch_status();
    }
    hipLaunchKernelGGL(sha256_batch_kernel, dim3(grid), dim3(256), 0, st, dev_recs, n);
    return launch_status();
}

}  // namespace aesctr
