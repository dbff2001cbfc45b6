// ctr_pair.hip -- AES-CTR of a message with about a block per lane (gfx950): two
// lanes per block.
//
// Between the sizes whose blocks get four lanes each (ctr_quad.hip) and those that
// fill the chip with a block per lane, the rounds run with one wave per SIMD: 16
// lookups and 28 VALU instructions in a chain with nothing beside it.  Here a pair
// of lanes holds a block, lane c columns 2c and 2c + 1, as two waves per SIMD with
// half the chain each: 8 lookups, 16 VALU instructions (two of them DPP moves) a
// round.  A workgroup is eight waves over 64 KiB of table copies, one per CU up to
// 1 MiB on 256 CUs.  What is left is the launch (1.56 us), the fill (about 0.5)
// and 9 rounds of 24 instructions on two waves (0.7).
//
// The keys reach the lanes through LDS, read before the tables, so that the
// fill's waits cover neither them nor the message (with the keys' loads last it
// waited for both: 1 MiB 3.06 us; with the message behind the fill, 2.86).
// Measured per launch in a replayed graph, against one lane per block: AES-128,
// 640 KiB 2.69 us (3.28), 1 MiB 2.79 (3.26); AES-256, 3.04 (3.74), 3.12 (3.81).
// Batches of a few requests of this size in all take the same path
// (ctr_pair_batch_kernel; figures at launch_small in batch.cpp).
#include "ttable_device.h"

namespace aesctr {
namespace {

constexpr int kPairWG = 512;
constexpr uint32_t kBlocks = kPairWG / 2;   // per workgroup
static_assert(kBlocks == kPairTileBlocks, "the tile of a small batch");

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(1)));
typedef __attribute__((address_space(1))) const u32x2_any g_cu32x2;
typedef __attribute__((address_space(1))) u32x2_any g_u32x2;

__constant__ u32x2 g_dummy;   // for the loads of a message of less than half a block

// The other lane's word.
__device__ __forceinline__ uint32_t other(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0xb1, 0xf, 0xf, true));
}

// A column of a round from the columns it reads (j, j + 1, j + 2, j + 3).
__device__ __forceinline__ uint32_t column(const TTable<kLayout2x32> &tt, uint32_t s0, uint32_t s1, uint32_t s2,
                                           uint32_t s3, uint32_t krot)
{
    return xor3(tt.raw<0, 0>(s0), tt.raw<1, 2>(s2), rotl8(xor3(tt.raw<0, 1>(s1), tt.raw<1, 3>(s3), krot)));
}

// Of the last round: T0 holds S in bytes 1 and 2, T2 in bytes 0 and 3.
__device__ __forceinline__ uint32_t last_column(const TTable<kLayout2x32> &tt, uint32_t s0, uint32_t s1, uint32_t s2,
                                                uint32_t s3, uint32_t k)
{
    return xor3(vperm(tt.raw<0, 1>(s1), tt.raw<1, 0>(s0), 0x0c0c0500u),
                vperm(tt.raw<1, 3>(s3), tt.raw<0, 2>(s2), 0x07020c0cu), k);
}

// Whether this lane has all of its half block at byte `at` of a message of len, or the
// bytes it has of it; the loads of the lanes without all go to valid memory.  (One
// yes or no for load and store: a byte count tested at both ends becomes a chain
// of branches at the store, 1 MiB 2.82 us instead of 2.76.)
__device__ __forceinline__ bool pair_whole(uint64_t at, uint64_t len) { return at + 8 <= len; }

__device__ __forceinline__ uint32_t pair_rest(uint64_t at, uint64_t len)
{
    return at < len ? static_cast<uint32_t>(len - at) : 0;
}

__device__ __forceinline__ u32x2 pair_load(const uint8_t *in, uint64_t at, uint64_t len, bool whole)
{
    g_cu8 *p = len >= 8 ? (g_cu8 *)in + (whole ? at : 0) : (g_cu8 *)&g_dummy;
    return __builtin_nontemporal_load((g_cu32x2 *)p);
}

__device__ __forceinline__ u32x2 pair_load_rest(const uint8_t *in, uint64_t at, uint64_t len, bool whole, u32x2 d)
{
    if (!whole) {
        const uint32_t have = pair_rest(at, len);
        g_cu8 *p = (g_cu8 *)in + at;
        d = u32x2{0, 0};
#pragma unroll
        for (uint32_t i = 0; i < 7; ++i)
            if (i < have)
                d[i >> 2] |= static_cast<uint32_t>(p[i]) << (8 * (i & 3));
    }
    return d;
}

__device__ __forceinline__ void pair_store(uint8_t *out, uint64_t at, uint64_t len, bool whole, u32x2 d)
{
    g_u8 *p = (g_u8 *)out + at;
    if (whole) {
        __builtin_nontemporal_store((u32x2_any)d, (g_u32x2 *)p);
    } else {
        const uint32_t have = pair_rest(at, len);
#pragma unroll
        for (uint32_t i = 0; i < 7; ++i)
            if (i < have)
                p[i] = static_cast<uint8_t>(d[i >> 2] >> (8 * (i & 3)));
    }
}

// Key word `lane` as it goes to LDS: those of the inner rounds rotated for the
// two-table fold.
__device__ __forceinline__ uint32_t pair_key(uint32_t kw, uint32_t lane, uint32_t nr)
{
    return lane >= 4 && lane < 4 + 4 * nr ? rotr8(kw) : kw;
}

// The lane's keys of rounds 1 (k1) .. NR from the key material (pair_key) from word
// 2c on.  Apart from the rounds because they go ahead of pair_load_rest: behind
// its branch, every launch of 1 MiB takes 2.85 us instead of 2.82.
template <int NR>
__device__ __forceinline__ void pair_keys(const u32x2 *ks, u32x2 (&k)[NR + 1])
{
    k[1] = ks[0];
#pragma unroll
    for (int r = 2; r <= NR; ++r) k[r] = ks[2 + 2 * r];
}

// Words 2c and 2c + 1 of the keystream block of counter ctr.
template <int NR>
__device__ __forceinline__ u32x2 pair_keystream(const TTable<kLayout2x32> &tt, const u32x2 (&k)[NR + 1], uint32_t c,
                                                uint32_t ctr, uint32_t x0)
{
    // Rounds 0 and 1: column j takes byte 3 - j of the counter column, by table 3 - j.
    const uint32_t x = vperm(ctr, ctr, 0x00010203u) ^ x0;    // big-endian counter
    const uint32_t lb = tt.lb0 + (c ? 0 : 128);              // T2 for columns 0 and 1
    uint32_t a = k[1][0] ^ rotl8(lds_at(tt.lds, (__builtin_amdgcn_ubfe(x, c ? 8 : 24, 8) << 8) + lb));
    uint32_t b = k[1][1] ^ lds_at(tt.lds, (__builtin_amdgcn_ubfe(x, c ? 0 : 16, 8) << 8) + lb);
#pragma unroll
    for (int r = 2; r < NR; ++r) {
        const uint32_t oa = other(a), ob = other(b);
        const uint32_t na = column(tt, a, b, oa, ob, k[r][0]);
        b = column(tt, b, oa, ob, a, k[r][1]);
        a = na;
    }
    const uint32_t oa = other(a), ob = other(b);
    return u32x2{last_column(tt, a, b, oa, ob, k[NR][0]), last_column(tt, b, oa, ob, a, k[NR][1])};
}

template <int NR>
__global__ __launch_bounds__(kPairWG) void ctr_pair_kernel(const uint8_t *in, uint8_t *out, uint64_t len, uint32_t ctr0,
                                                           uint32_t x0, const CtrKeys keys)
{
    __shared__ uint32_t lds[layout_lds_words(kLayout2x32)];
    __shared__ u32x2 lkeys[kPairWG / 2];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 1;
    const uint32_t kw = key_word(lane);
    uint32_t tv[kFillStores / kPairWG];
    fill_read<kLayout2x32, kPairWG>(tv);
    const uint64_t blk = static_cast<uint64_t>(blockIdx.x) * kBlocks + (threadIdx.x >> 1);
    const uint64_t at = 16 * blk + 8 * c;
    const bool whole = pair_whole(at, len);
    u32x2 d = pair_load(in, at, len, whole);
    __builtin_amdgcn_sched_barrier(0);

    fill_write<kLayout2x32, kPairWG>(lds, tv);
    reinterpret_cast<uint32_t *>(lkeys)[threadIdx.x] = pair_key(kw, lane, NR);   // each wave for itself
    __syncthreads();
    u32x2 k[NR + 1];
    pair_keys<NR>(lkeys + 32 * wave + c, k);
    d = pair_load_rest(in, at, len, whole, d);
    const TTable<kLayout2x32> tt{reinterpret_cast<const char *>(lds), 4 * (lane & 31), 0};
    d ^= pair_keystream<NR>(tt, k, c, ctr0 + static_cast<uint32_t>(blk), x0);
    pair_store(out, at, len, whole, d);
}

// A few requests whose records travel in the kernel argument block
// (SmallBatchArgs, tile_blocks = kBlocks): workgroup t takes tile t.
__global__ __launch_bounds__(kPairWG) void ctr_pair_batch_kernel(const SmallBatchArgs args)
{
    __shared__ uint32_t lds[layout_lds_words(kLayout2x32)];
    __shared__ u32x2 lkeys[kPairWG / 2];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 1, t = blockIdx.x;
    uint32_t tv[kFillStores / kPairWG];
    fill_read<kLayout2x32, kPairWG>(tv);
    const uint32_t n = args.n;
    // Last request whose first tile is <= t (skips empty requests).
    uint32_t r = 0;
#pragma unroll
    for (uint32_t i = 1; i < kSmallBatch; ++i)
        if (i < n && args.r[i].tile0 <= t)
            r = i;
    const SmallRec &R = args.r[r];
    uint32_t *resident = reinterpret_cast<uint32_t *>(args.resident);
    uint32_t kw = 0;
    if (lane < 4)
        kw = R.k1[lane];
    else if (R.key & kKeyResident)
        kw = resident[64u * (R.key & ~kKeyResident) + lane - 4];
    else
        kw = R.rk[lane - 4];
    const uint8_t *in = reinterpret_cast<const uint8_t *>(R.in);
    uint8_t *out = reinterpret_cast<uint8_t *>(R.out);
    const uint64_t len = R.len;
    const uint64_t blk = static_cast<uint64_t>(t - R.tile0) * kBlocks + (threadIdx.x >> 1);
    const uint64_t at = 16 * blk + 8 * c;
    const bool whole = pair_whole(at, len);
    const uint32_t ctr = R.ctr0 + static_cast<uint32_t>(blk), x0 = R.x0, nr = R.nr;
    u32x2 d = pair_load(in, at, len, whole);
    fill_write<kLayout2x32, kPairWG>(lds, tv);
    reinterpret_cast<uint32_t *>(lkeys)[threadIdx.x] = pair_key(kw, lane, nr);
    __syncthreads();
    d = pair_load_rest(in, at, len, whole, d);
    const TTable<kLayout2x32> tt{reinterpret_cast<const char *>(lds), 4 * (lane & 31), 0};
    const u32x2 *ks = lkeys + 32 * wave + c;
    if (nr == 10) {
        u32x2 k[11];
        pair_keys<10>(ks, k);
        d ^= pair_keystream<10>(tt, k, c, ctr, x0);
    } else {
        u32x2 k[15];
        pair_keys<14>(ks, k);
        d ^= pair_keystream<14>(tt, k, c, ctr, x0);
    }
    pair_store(out, at, len, whole, d);
    // No wave of this launch reads a slot that it installs.
    if (t == 0) {
        for (uint32_t j = threadIdx.x; j < 64u * n; j += kPairWG) {
            const uint32_t i = j >> 6, w = j & 63u;
            if (args.r[i].install != kNoInstall && w < 60u)
                resident[64u * args.r[i].install + w] = args.r[i].rk[w];
        }
    }
}

template <int NR>
void launch_pair(const CtrArgs &a, hipStream_t st)
{
    const uint64_t blocks = (a.len + 15) / 16;
    const dim3 grid(static_cast<uint32_t>((blocks + kBlocks - 1) / kBlocks));
    hipLaunchKernelGGL(ctr_pair_kernel<NR>, grid, dim3(kPairWG), 0, st, a.in, a.out, a.len, a.ctr0, a.x0, ctr_keys(a));
}

}  // namespace

// From where quads of lanes stop (quad_shape is asked first) to 256 blocks per CU,
// one workgroup each: a second one on a CU would fill its tables again and run
// beside the first.  Pairs against one lane per block, AES-128 and AES-256: 1 MiB
// 2.79 us against 3.26 and 3.12 against 3.81; 1.1 MB 3.85 against 3.45 and 4.37
// against 4.06.  Against quads: 512 KiB 2.73 against 2.44, 800,000 bytes 2.78
// against 3.18.  Asked for calls that name no shape, as quad_shape is.
bool pair_shape(const Shape &sh, uint64_t len, int num_cus)
{
    const uint64_t blocks = (len + 15) / 16;
    return sh.copies == 32 && sh.tables == 2 && sh.wg == 256 && sh.bpl == 1 && sh.wave_groups == kFirstFull &&
           blocks <= 256 * static_cast<uint64_t>(num_cus) && blocks <= static_cast<uint64_t>(sh.grid) * sh.wg;
}

int launch_ctr_pair(const CtrArgs &a, int nr, hipStream_t st)
{
    (void)hipGetLastError();   // not ours: left by earlier calls
    if (nr == 10)
        launch_pair<10>(a, st);
    else if (nr == 14)
        launch_pair<14>(a, st);
    else
        return AES_EINVAL;
    return launch_status();
}

int launch_ctr_pair_batch(const SmallBatchArgs &args, hipStream_t st)
{
    if (args.n > kSmallBatch || args.tile_blocks != kPairTileBlocks || args.total_tiles == 0 ||
        args.total_tiles > 0x7fffffffu)
        return AES_EINVAL;
    (void)hipGetLastError();   // not ours: left by earlier calls
    hipLaunchKernelGGL(ctr_pair_batch_kernel, dim3(args.total_tiles), dim3(kPairWG), 0, st, args);
    return launch_status();
}

}  // namespace aesctr
