// ctr_quad.hip -- AES-CTR of a small message (gfx950): four lanes per block.
//
// A message of up to a few hundred KiB has fewer blocks than the chip has lanes,
// so its time is the chain of one block's rounds.  Here a quad of lanes holds a
// block, lane c column c: a round is 4 lookups, 4 address operations, 3 DPP moves
// and 2 XORs per lane, where one lane per block (ctr_ttable.hip) does 16 lookups
// and 28 VALU instructions in a row.  A workgroup is one wave with one copy of the
// four round tables (4 KiB of LDS): the random lookups of a wave meet in the banks
// three or four deep, which costs less here than filling 64 KiB of copies.
// (Sixteen waves of quads over 64 KiB of copies: 2.68 us at 4 KiB and 3.16 us at
// 512 KiB, between the two everywhere, so not kept.)
// Measured per launch in a replayed graph, AES-128, against one lane per block:
// 4 KiB 1.93 us (2.89), 64 KiB 2.08 (3.08), 256 KiB 2.60 (3.14), 512 KiB 2.96 (3.19);
// AES-256: 2.35 (3.40), 2.58 (3.58), 2.82 (3.63), 3.31 (3.71).  An empty launch takes
// 1.56 us there; the rest is the table and message reads and the chain of rounds.
#include "ttable_device.h"

namespace aesctr {
namespace {

// The key material as the lanes read it, a column each, from the kernel's
// argument block (CtrKeys lies behind the scalars).
constexpr size_t kKeysOffset = 32;
typedef const __attribute__((address_space(4))) uint32_t c_u32;

constexpr uint32_t kBlocks = 16;   // per wave, which is a workgroup

template <int CTRL>
__device__ __forceinline__ uint32_t quad(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xf, 0xf, true));
}

template <int NR>
__global__ __launch_bounds__(64) void ctr_quad_kernel(const uint8_t *in, uint8_t *out, uint64_t len, uint32_t ctr0,
                                                      uint32_t x0, const CtrKeys keys)
{
    static_assert(sizeof(void *) * 2 + sizeof(uint64_t) + 2 * sizeof(uint32_t) == kKeysOffset, "argument layout");
    __shared__ uint32_t lds[4 * 256];   // table t at word 256 t
    const uint32_t lane = threadIdx.x, c = lane & 3;
    const u32x4 t0 = reinterpret_cast<const u32x4 *>(c_round.t[0])[lane];

    // This lane's word of its block; of the last, partial block the bytes there are.
    const uint64_t blk = static_cast<uint64_t>(blockIdx.x) * kBlocks + (lane >> 2);
    const uint64_t at = 16 * blk + 4 * c;
    const uint32_t have = at + 4 <= len ? 4 : at < len ? static_cast<uint32_t>(len - at) : 0;
    g_cu8 *src = (g_cu8 *)in + at;
    uint32_t d = 0;
    if (have == 4) {
        d = __builtin_nontemporal_load((g_cu32 *)src);
    } else {
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i)
            if (i < have)
                d |= static_cast<uint32_t>(src[i]) << (8 * i);
    }
    c_u32 *kp = (c_u32 *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() +
                          kKeysOffset) + c;
    const uint32_t k1 = kp[0];
    uint32_t rk[NR + 1];
#pragma unroll
    for (int r = 2; r <= NR; ++r) rk[r] = kp[4 + 4 * r];

#pragma unroll
    for (int t = 0; t < 4; ++t) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_alignbit(t0[i], t0[i], (32 - 8 * t) & 31);
        *reinterpret_cast<u32x4 *>(&lds[256 * t + 4 * lane]) = v;
    }
    __syncthreads();

    // Rounds 0 and 1: column c takes byte 3 - c of the counter column.
    const uint32_t ctr = ctr0 + static_cast<uint32_t>(blk);
    const uint32_t x = vperm(ctr, ctr, 0x00010203u) ^ x0;    // big-endian counter
    uint32_t s = k1 ^ lds[256 * (3 - c) + __builtin_amdgcn_ubfe(x, 24 - 8 * c, 8)];
#pragma unroll
    for (int r = 2; r < NR; ++r) {
        const uint32_t s1 = quad<0x39>(s), s2 = quad<0x4e>(s), s3 = quad<0x93>(s);   // columns c + 1, 2, 3
        s = xor3(xor3(lds[s & 255u], lds[256 + ((s1 >> 8) & 255u)], lds[512 + ((s2 >> 16) & 255u)]),
                 lds[768 + (s3 >> 24)], rk[r]);
    }
    // The last round's S bytes: T0 holds S in bytes 1 and 2, T2 in bytes 0 and 3.
    const uint32_t s1 = quad<0x39>(s), s2 = quad<0x4e>(s), s3 = quad<0x93>(s);
    const uint32_t lo = vperm(lds[(s1 >> 8) & 255u], lds[512 + (s & 255u)], 0x0c0c0500u);
    const uint32_t hi = vperm(lds[512 + (s3 >> 24)], lds[(s2 >> 16) & 255u], 0x07020c0cu);
    d ^= xor3(lo, hi, rk[NR]);

    g_u8 *dst = (g_u8 *)out + at;
    if (have == 4) {
        __builtin_nontemporal_store(d, (g_u32 *)dst);
    } else {
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i)
            if (i < have)
                dst[i] = static_cast<uint8_t>(d >> (8 * i));
    }
}

template <int NR>
void launch_quad(const CtrArgs &a, hipStream_t st)
{
    const uint64_t blocks = (a.len + 15) / 16;
    const dim3 grid(static_cast<uint32_t>((blocks + kBlocks - 1) / kBlocks));
    hipLaunchKernelGGL(ctr_quad_kernel<NR>, grid, dim3(64), 0, st, a.in, a.out, a.len, a.ctr0, a.x0, ctr_keys(a));
}

}  // namespace

// Up to 128 blocks per CU (512 KiB on 256 CUs), two waves of quads per SIMD: from
// there the bank conflicts of the one table copy cost what the shorter chain
// saves.  Quads against one lane per block, AES-128 and AES-256: 512 KiB 2.96 us
// against 3.19 and 3.31 against 3.71; 700,001 bytes 3.28 against 3.29 and 3.81
// against 3.73; 1 MiB 3.82 against 3.26 and 4.52 against 3.80.  A grid that is
// smaller than the work is the caller's choice and is kept.
bool quad_shape(const Shape &sh, uint64_t len, int num_cus)
{
    const uint64_t blocks = (len + 15) / 16;
    return sh.copies == 32 && sh.tables == 2 && sh.wg == 256 && sh.bpl == 1 && sh.wave_groups == kFirstFull &&
           blocks <= 128 * static_cast<uint64_t>(num_cus) && blocks <= static_cast<uint64_t>(sh.grid) * sh.wg;
}

int launch_ctr_quad(const CtrArgs &a, int nr, hipStream_t st)
{
    (void)hipGetLastError();   // not ours: left by earlier calls
    if (nr == 10)
        launch_quad<10>(a, st);
    else if (nr == 14)
        launch_quad<14>(a, st);
    else
        return AES_EINVAL;
    return launch_status();
}

}  // namespace aesctr
