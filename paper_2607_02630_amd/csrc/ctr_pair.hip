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
#include "ttable_device.h"

namespace aesctr {
namespace {

constexpr int kPairWG = 512;
constexpr uint32_t kBlocks = kPairWG / 2;   // per workgroup

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

    // This lane's half of its block; of the last, partial block the bytes there are.
    const uint64_t blk = static_cast<uint64_t>(blockIdx.x) * kBlocks + (threadIdx.x >> 1);
    const uint64_t at = 16 * blk + 8 * c;
    const uint32_t have = at + 8 <= len ? 8 : at < len ? static_cast<uint32_t>(len - at) : 0;
    g_cu8 *src = (g_cu8 *)in + at;
    g_cu8 *whole = len >= 8 ? (g_cu8 *)in + (have == 8 ? at : 0) : (g_cu8 *)&g_dummy;
    u32x2 d = __builtin_nontemporal_load((g_cu32x2 *)whole);
    __builtin_amdgcn_sched_barrier(0);

    // Each wave keeps the keys for itself, those of the inner rounds rotated for
    // the two-table fold.
    fill_write<kLayout2x32, kPairWG>(lds, tv);
    reinterpret_cast<uint32_t *>(lkeys)[threadIdx.x] = lane >= 4 && lane < 4 + 4 * NR ? rotr8(kw) : kw;
    __syncthreads();

    const u32x2 *ks = lkeys + 32 * wave + c;
    const u32x2 k1 = ks[0];
    u32x2 rk[NR + 1];
#pragma unroll
    for (int r = 2; r <= NR; ++r) rk[r] = ks[2 + 2 * r];
    if (have < 8) {
        d = u32x2{0, 0};
#pragma unroll
        for (uint32_t i = 0; i < 7; ++i)
            if (i < have)
                d[i >> 2] |= static_cast<uint32_t>(src[i]) << (8 * (i & 3));
    }

    // Rounds 0 and 1: column j takes byte 3 - j of the counter column, by table 3 - j.
    const TTable<kLayout2x32> tt{reinterpret_cast<const char *>(lds), 4 * (lane & 31), 0};
    const uint32_t ctr = ctr0 + static_cast<uint32_t>(blk);
    const uint32_t x = vperm(ctr, ctr, 0x00010203u) ^ x0;    // big-endian counter
    const uint32_t lb = tt.lb0 + (c ? 0 : 128);              // T2 for columns 0 and 1
    uint32_t a = k1[0] ^ rotl8(lds_at(tt.lds, (__builtin_amdgcn_ubfe(x, c ? 8 : 24, 8) << 8) + lb));
    uint32_t b = k1[1] ^ lds_at(tt.lds, (__builtin_amdgcn_ubfe(x, c ? 0 : 16, 8) << 8) + lb);
#pragma unroll
    for (int r = 2; r < NR; ++r) {
        const uint32_t oa = other(a), ob = other(b);
        const uint32_t na = column(tt, a, b, oa, ob, rk[r][0]);
        b = column(tt, b, oa, ob, a, rk[r][1]);
        a = na;
    }
    const uint32_t oa = other(a), ob = other(b);
    d[0] ^= last_column(tt, a, b, oa, ob, rk[NR][0]);
    d[1] ^= last_column(tt, b, oa, ob, a, rk[NR][1]);

    g_u8 *dst = (g_u8 *)out + at;
    if (have == 8) {
        __builtin_nontemporal_store((u32x2_any)d, (g_u32x2 *)dst);
    } else {
#pragma unroll
        for (uint32_t i = 0; i < 7; ++i)
            if (i < have)
                dst[i] = static_cast<uint8_t>(d[i >> 2] >> (8 * (i & 3)));
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
// against 3.18.  A grid that is smaller than the work is the caller's choice and is kept.
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

}  // namespace aesctr
