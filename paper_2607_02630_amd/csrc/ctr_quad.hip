// ctr_quad.hip -- AES-CTR of a small message (gfx950): four lanes per block.
//
// A message of up to a few hundred KiB has fewer blocks than the chip has lanes,
// so its time is the chain of one block's rounds.  Here a quad of lanes holds a
// block, lane c column c: a round is 4 lookups, 4 address operations, 3 DPP moves
// and 2 XORs per lane, where one lane per block (ctr_ttable.hip) does 16 lookups
// and 28 VALU instructions in a row.  A workgroup is four waves with one copy of
// the four round tables (4 KiB of LDS, a table per wave to write): the random
// lookups of a wave meet in the banks about three deep, which costs less here
// than filling 64 KiB of copies.  (Sixteen waves of quads over 64 KiB of copies:
// 2.68 us at 4 KiB and 3.16 us at 512 KiB.)
//
// The keys reach the lanes through LDS (key_word), and the message is asked for
// behind the table's stores: no wait of the fill then covers it, and the table
// reads of 2048 waves don't queue behind it.  The keys loaded per lane from the
// argument block and the message first, one wave per workgroup: 2.57 us at 256
// KiB, 2.96 us at 512 KiB; keys through LDS and the message last: 2.16, 2.80; four
// waves per workgroup: 2.07, 2.44 (and 1.90 instead of 1.80 at 16 bytes).
// Measured per launch in a replayed graph, AES-128, against one lane per block:
// 4 KiB 1.92 us (2.89), 64 KiB 2.02 (3.08), 256 KiB 2.07 (3.14), 512 KiB 2.44 (3.19);
// AES-256: 2.13 (3.40), 2.21 (3.58), 2.29 (3.63), 2.80 (3.71).  An empty launch takes
// 1.56 us there.  Batches of a few small requests take the same path
// (ctr_quad_batch_kernel, ctr_quad_table_kernel; figures at launch_small and
// quad_table in batch.cpp).
#include "ttable_device.h"

namespace aesctr {
namespace {

constexpr uint32_t kQuadWG = 256;
constexpr uint32_t kBlocks = kQuadWG / 4;   // per workgroup
static_assert(kBlocks == kQuadTileBlocks, "the tile of a small batch");

__constant__ uint32_t g_dummy;   // for the loads of a message of less than a word

template <int CTRL>
__device__ __forceinline__ uint32_t quad(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xf, 0xf, true));
}

// The table of this wave from T0's entries 4 lane .. 4 lane + 3: T0 rotated.
__device__ __forceinline__ void quad_fill(uint32_t *lds, u32x4 t0, uint32_t wave, uint32_t lane)
{
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_alignbit(t0[i], t0[i], (32 - 8 * wave) & 31);
    *reinterpret_cast<u32x4 *>(&lds[256 * wave + 4 * lane]) = v;
}

// Whether this lane has all of its word at byte `at` of a message of len, or the
// bytes it has of it; the loads of the lanes without all go to valid memory.
__device__ __forceinline__ bool quad_whole(uint64_t at, uint64_t len) { return at + 4 <= len; }

__device__ __forceinline__ uint32_t quad_rest(uint64_t at, uint64_t len)
{
    return at < len ? static_cast<uint32_t>(len - at) : 0;
}

__device__ __forceinline__ uint32_t quad_load(const uint8_t *in, uint64_t at, uint64_t len, bool whole)
{
    g_cu8 *p = len >= 4 ? (g_cu8 *)in + (whole ? at : 0) : (g_cu8 *)&g_dummy;
    return __builtin_nontemporal_load((g_cu32 *)p);
}

__device__ __forceinline__ uint32_t quad_load_rest(const uint8_t *in, uint64_t at, uint64_t len, bool whole, uint32_t d)
{
    if (!whole) {
        const uint32_t have = quad_rest(at, len);
        g_cu8 *p = (g_cu8 *)in + at;
        d = 0;
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i)
            if (i < have)
                d |= static_cast<uint32_t>(p[i]) << (8 * i);
    }
    return d;
}

__device__ __forceinline__ void quad_store(uint8_t *out, uint64_t at, uint64_t len, bool whole, uint32_t d)
{
    g_u8 *p = (g_u8 *)out + at;
    if (whole) {
        __builtin_nontemporal_store(d, (g_u32 *)p);
    } else {
        const uint32_t have = quad_rest(at, len);
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i)
            if (i < have)
                p[i] = static_cast<uint8_t>(d >> (8 * i));
    }
}

// The lane's keys of rounds 1 (k1) .. NR from the key material (CtrKeys) from word c on.
template <int NR>
__device__ __forceinline__ void quad_keys(const uint32_t *ks, uint32_t (&k)[NR + 1])
{
    k[1] = ks[0];
#pragma unroll
    for (int r = 2; r <= NR; ++r) k[r] = ks[4 + 4 * r];
}

// Word c of the keystream block of counter ctr.
template <int NR>
__device__ __forceinline__ uint32_t quad_keystream(const uint32_t *lds, const uint32_t (&k)[NR + 1], uint32_t c,
                                                   uint32_t ctr, uint32_t x0)
{
    // Rounds 0 and 1: column c takes byte 3 - c of the counter column.
    const uint32_t x = vperm(ctr, ctr, 0x00010203u) ^ x0;    // big-endian counter
    uint32_t s = k[1] ^ lds[256 * (3 - c) + __builtin_amdgcn_ubfe(x, 24 - 8 * c, 8)];
#pragma unroll
    for (int r = 2; r < NR; ++r) {
        const uint32_t s1 = quad<0x39>(s), s2 = quad<0x4e>(s), s3 = quad<0x93>(s);   // columns c + 1, 2, 3
        s = xor3(xor3(lds[s & 255u], lds[256 + ((s1 >> 8) & 255u)], lds[512 + ((s2 >> 16) & 255u)]),
                 lds[768 + (s3 >> 24)], k[r]);
    }
    // The last round's S bytes: T0 holds S in bytes 1 and 2, T2 in bytes 0 and 3.
    const uint32_t s1 = quad<0x39>(s), s2 = quad<0x4e>(s), s3 = quad<0x93>(s);
    const uint32_t lo = vperm(lds[(s1 >> 8) & 255u], lds[512 + (s & 255u)], 0x0c0c0500u);
    const uint32_t hi = vperm(lds[512 + (s3 >> 24)], lds[(s2 >> 16) & 255u], 0x07020c0cu);
    return xor3(lo, hi, k[NR]);
}

template <int NR>
__global__ __launch_bounds__(kQuadWG) void ctr_quad_kernel(const uint8_t *in, uint8_t *out, uint64_t len, uint32_t ctr0,
                                                           uint32_t x0, const CtrKeys keys)
{
    __shared__ uint32_t lds[4 * 256];   // table t at word 256 t
    __shared__ uint32_t lkeys[kQuadWG];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 3;
    const u32x4 t0 = reinterpret_cast<const u32x4 *>(c_round.t[0])[lane];
    const uint32_t kw = key_word(lane);
    __builtin_amdgcn_sched_barrier(0);
    quad_fill(lds, t0, wave, lane);
    lkeys[threadIdx.x] = kw;            // each wave for itself
    __builtin_amdgcn_sched_barrier(0);

    const uint64_t blk = static_cast<uint64_t>(blockIdx.x) * kBlocks + (threadIdx.x >> 2);
    const uint64_t at = 16 * blk + 4 * c;
    const bool whole = quad_whole(at, len);
    uint32_t d = quad_load(in, at, len, whole);
    __syncthreads();
    uint32_t k[NR + 1];
    quad_keys<NR>(lkeys + 64 * wave + c, k);
    d = quad_load_rest(in, at, len, whole, d);
    d ^= quad_keystream<NR>(lds, k, c, ctr0 + static_cast<uint32_t>(blk), x0);
    quad_store(out, at, len, whole, d);
}

// A lane's word d of a request of either key size, whose key material from word c on
// is ks (quad_keys), from behind its load to its store.
__device__ __forceinline__ void quad_crypt(const uint32_t *lds, const uint32_t *ks, uint32_t c, const uint8_t *in,
                                           uint8_t *out, uint64_t at, uint64_t len, bool whole, uint32_t d,
                                           uint32_t ctr, uint32_t x0, uint32_t nr)
{
    d = quad_load_rest(in, at, len, whole, d);
    if (nr == 10) {
        uint32_t k[11];
        quad_keys<10>(ks, k);
        d ^= quad_keystream<10>(lds, k, c, ctr, x0);
    } else {
        uint32_t k[15];
        quad_keys<14>(ks, k);
        d ^= quad_keystream<14>(lds, k, c, ctr, x0);
    }
    quad_store(out, at, len, whole, d);
}

// A few small requests whose records travel in the kernel argument block
// (SmallBatchArgs, tile_blocks = kBlocks): workgroup t takes tile t.
__global__ __launch_bounds__(kQuadWG) void ctr_quad_batch_kernel(const SmallBatchArgs args)
{
    __shared__ uint32_t lds[4 * 256];
    __shared__ uint32_t lkeys[kQuadWG];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 3, t = blockIdx.x;
    const u32x4 t0 = reinterpret_cast<const u32x4 *>(c_round.t[0])[lane];
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
    const uint64_t blk = static_cast<uint64_t>(t - R.tile0) * kBlocks + (threadIdx.x >> 2);
    const uint64_t at = 16 * blk + 4 * c;
    const bool any = t < args.total_tiles;     // no tile at all: a launch for its installs
    const uint64_t len = any ? R.len : 0;
    const bool whole = quad_whole(at, len);
    const uint32_t ctr = R.ctr0 + static_cast<uint32_t>(blk), x0 = R.x0, nr = R.nr;
    uint8_t *out = reinterpret_cast<uint8_t *>(R.out);
    quad_fill(lds, t0, wave, lane);
    lkeys[threadIdx.x] = kw;
    uint32_t d = quad_load(in, at, len, whole);
    __syncthreads();
    if (any)
        quad_crypt(lds, lkeys + 64 * wave + c, c, in, out, at, len, whole, d, ctr, x0, nr);
    // No wave of this launch reads a slot that it installs.
    if (t == 0) {
        for (uint32_t j = threadIdx.x; j < 64u * n; j += kQuadWG) {
            const uint32_t i = j >> 6, w = j & 63u;
            if (args.r[i].install != kNoInstall && w < 60u)
                resident[64u * args.r[i].install + w] = args.r[i].rk[w];
        }
    }
}

// More requests than the argument block takes, as few blocks: records, keys and
// installs in the uploaded table.  The scalars of its header come as arguments,
// and a wave finds its request by counting the first tiles up to t, a request
// per lane and load: one memory round trip each for them, the request and the key.
__global__ __launch_bounds__(kQuadWG) void ctr_quad_table_kernel(const uint8_t *__restrict__ table, uint32_t *resident,
                                                                 uint32_t n, uint32_t total, uint32_t n_install,
                                                                 uint32_t install_off)
{
    __shared__ uint32_t lds[4 * 256];
    __shared__ uint32_t lkeys[kQuadWG];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 3, t = blockIdx.x;
    const BatchDesc *desc = reinterpret_cast<const BatchDesc *>(table + sizeof(BatchHeader));
    const uint32_t *keys = reinterpret_cast<const uint32_t *>(table + batch_keys_off(n));
    uint32_t first[kQuadTableReqs / 64];
#pragma unroll
    for (uint32_t u = 0; u < kQuadTableReqs / 64; ++u) {
        const uint32_t i = lane + 64 * u;
        first[u] = desc[i < n ? i : n - 1].tile0;
    }
    const u32x4 t0 = reinterpret_cast<const u32x4 *>(c_round.t[0])[lane];
    // Last request whose first tile is <= t: tile0 ascends from 0, and empty
    // requests share their successor's.
    uint32_t upto = 0;
#pragma unroll
    for (uint32_t u = 0; u < kQuadTableReqs / 64; ++u)
        upto += static_cast<uint32_t>(__popcll(__ballot(lane + 64 * u < n && first[u] <= t)));
    const BatchDesc &R = desc[__builtin_amdgcn_readfirstlane(upto) - 1];
    const uint32_t key = R.key;
    const uint32_t *from = key & kKeyResident ? resident + 64u * (key & ~kKeyResident) : keys + 64u * key;
    const uint32_t kw = lane < 4 ? R.k1[lane] : from[lane - 4];
    const uint8_t *in = reinterpret_cast<const uint8_t *>(R.in);
    uint8_t *out = reinterpret_cast<uint8_t *>(R.out);
    const uint64_t blk = static_cast<uint64_t>(t - R.tile0) * kBlocks + (threadIdx.x >> 2);
    const uint64_t at = 16 * blk + 4 * c;
    const bool any = t < total;     // no tile at all: a launch for its installs
    const uint64_t len = any ? R.len : 0;
    const bool whole = quad_whole(at, len);
    const uint32_t ctr = R.ctr0 + static_cast<uint32_t>(blk), x0 = R.x0, nr = R.nr;
    quad_fill(lds, t0, wave, lane);
    lkeys[threadIdx.x] = kw;
    uint32_t d = quad_load(in, at, len, whole);
    __syncthreads();
    if (any)
        quad_crypt(lds, lkeys + 64 * wave + c, c, in, out, at, len, whole, d, ctr, x0, nr);
    // No wave of this launch reads a slot that it installs.
    if (t == 0) {
        const InstallRec *inst = reinterpret_cast<const InstallRec *>(table + install_off);
        for (uint32_t j = threadIdx.x; j < 64u * n_install; j += kQuadWG) {
            const InstallRec r = inst[j >> 6];
            resident[64u * r.slot + (j & 63u)] = keys[64u * r.key + (j & 63u)];
        }
    }
}

template <int NR>
void launch_quad(const CtrArgs &a, hipStream_t st)
{
    const uint64_t blocks = (a.len + 15) / 16;
    const dim3 grid(static_cast<uint32_t>((blocks + kBlocks - 1) / kBlocks));
    hipLaunchKernelGGL(ctr_quad_kernel<NR>, grid, dim3(kQuadWG), 0, st, a.in, a.out, a.len, a.ctr0, a.x0, ctr_keys(a));
}

}  // namespace

// Up to 128 blocks per CU (512 KiB on 256 CUs), two workgroups of quads: from
// there the bank conflicts of the one table copy cost what the shorter chain
// saves.  Quads against one lane per block, AES-128 and AES-256: 512 KiB 2.44 us
// against 3.19 and 2.80 against 3.71; 1 MiB 3.28 against 3.26 and 4.02 against 3.81.
// Asked for calls that name no shape; a tuned grid that is smaller than the work keeps its kernel.
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

int launch_ctr_quad_batch(const SmallBatchArgs &args, hipStream_t st)
{
    if (args.n > kSmallBatch || args.tile_blocks != kQuadTileBlocks || args.total_tiles > 0x7fffffffu)
        return AES_EINVAL;
    (void)hipGetLastError();   // not ours: left by earlier calls
    const dim3 grid(args.total_tiles ? args.total_tiles : 1);
    hipLaunchKernelGGL(ctr_quad_batch_kernel, grid, dim3(kQuadWG), 0, st, args);
    return launch_status();
}

int launch_ctr_quad_table(const void *dev_table, const BatchHeader &h, hipStream_t st)
{
    if (h.n == 0 || h.n > kQuadTableReqs || h.tile_blocks != kQuadTileBlocks || h.total_tiles > 0x7fffffffu)
        return AES_EINVAL;
    (void)hipGetLastError();   // not ours: left by earlier calls
    const dim3 grid(h.total_tiles ? h.total_tiles : 1);
    hipLaunchKernelGGL(ctr_quad_table_kernel, grid, dim3(kQuadWG), 0, st, static_cast<const uint8_t *>(dev_table),
                       reinterpret_cast<uint32_t *>(h.resident), h.n, h.total_tiles, h.n_install, h.install_off);
    return launch_status();
}

}  // namespace aesctr
