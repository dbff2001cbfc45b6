// ctr_bulk.hip -- AES-CTR of one large message (gfx950): T-tables in LDS, one
// persistent workgroup per CU whose waves take tiles from a counter in LDS.
//
// The round code, the four-table layout and the split of rounds 1-2 are those of
// ttable_device.h and ttable_tile.h.  A tile is 256 positions, one counter group
// (positions start at ctr0 mod 256, so the lanes' constants are the same for
// every tile and a tile has one set of group constants; a wave computes those of
// its workgroup's next 64 tiles at once, a lane each).
//
// Why waves take tiles instead of equal shares: the oldest wave of a SIMD wins
// the issue slot, so with equal shares the first waves of a workgroup end at 95
// of 155 us and the last work alone.
//
// Bound: 129.6 (AES-256: 193.6) table lookups and 215 (313) VALU instructions per
// block, counted; the LDS gives 26.5 (27.9) of the 32 lookups per clock and CU that
// its two clocks per instruction allow, at the 2.0-2.1 GHz the card holds under this
// load (2.4 without the payload traffic).
// Measured: 256 MiB AES-128 153 us = 1755 GB/s (167 before, two 512-thread
// workgroups with equal shares per CU), AES-256 208 us = 1290 GB/s (230); ragged
// 100 MB AES-256 in place 80 us (89).
#include "ttable_tile.h"

namespace aesctr {
namespace {

constexpr int kBulkWG = 1024;
constexpr int kBulkLayout = kLayout4x32;
constexpr uint32_t kBulkTile = 256;

template <int NR>
__global__ __launch_bounds__(kBulkWG) void ctr_bulk_kernel(const uint8_t *in, uint8_t *out, uint64_t len,
                                                           uint32_t ctr0, uint32_t x0, const CtrKeys keys)
{
    CtrArgs a;
    a.in = in;
    a.out = out;
    a.len = len;
    a.ctr0 = ctr0;
    a.x0 = x0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        a.k1[i] = keys.k1[i];
#pragma unroll
    for (int i = 0; i < 4 * (NR + 1); ++i)
        a.rk[i] = keys.rk[i];
    __shared__ uint32_t lds[layout_lds_words(kBulkLayout)];
    __shared__ uint32_t s_next;

    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t tv[kFillStores / kBulkWG];
    fill_read<kBulkLayout, kBulkWG>(tv);
    fill_write<kBulkLayout, kBulkWG>(lds, tv);
    if (threadIdx.x == 0)
        s_next = kBulkWG / 64;    // the waves' first tiles are their own numbers
    __syncthreads();
    const TTable<kBulkLayout> tt{reinterpret_cast<const char *>(lds), 4 * (lane & 31), 4 * (lane & 31) | 0x10000u};

    const uint32_t shift = a.ctr0 & 255u, tail = static_cast<uint32_t>(a.len & 15);
    const uint32_t tiles = static_cast<uint32_t>((shift + ((a.len + 15) >> 4) + kBulkTile - 1) / kBulkTile);
    const uint32_t grid = gridDim.x;
    uint32_t L[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        lane_consts(tt, a, 64 * k + lane, L[k]);
    uint32_t Gv[4];
    uint32_t window = ~0u;    // the 64 of the workgroup's tiles whose group constants Gv holds
    for (uint32_t j = wave;;) {
        const uint32_t t = j * grid + blockIdx.x;
        if (t >= tiles)
            break;
        uint32_t next = 0;
        if (lane == 0)
            next = atomicAdd(&s_next, 1u);
        const uint64_t p0 = static_cast<uint64_t>(t) * kBulkTile;
        const Span sp = message_span(a, shift, p0, p0 + kBulkTile);
        u32x4 part = {0, 0, 0, 0};
        if (sp.odd != ~0u)
            part = load_partial(sp.in, sp.odd, tail);
        if ((j >> 6) != window) {
            window = j >> 6;
            const uint32_t tl = ((window << 6) + lane) * grid + blockIdx.x;
            group_consts_lds(tt, a, ((a.ctr0 >> 8) + tl) & 0xffffffu, Gv);
        }
        uint32_t G[2][4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            G[0][c] = G[1][c] = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(Gv[c]), j & 63));
        span_step<NR, kBulkLayout, 2>(tt, a, nullptr, sp, 0, lane, &L[0], G, part);
        span_step<NR, kBulkLayout, 2>(tt, a, nullptr, sp, 128, lane, &L[2], G, part);
        if (sp.odd != ~0u && lane == (sp.odd & 63))
            store_partial(sp.out, sp.odd, tail, part);
        j = __builtin_amdgcn_readfirstlane(next);
    }
}

}  // namespace

bool bulk_shape(const Shape &sh, uint64_t len)
{
    return sh.copies == 32 && sh.tables == 4 && sh.wg == kBulkWG && sh.bpl == 2 && sh.wave_groups == kFirstWave0 &&
           len / 16 >= static_cast<uint64_t>(sh.grid) * (kBulkWG / 64) * kBulkTile;
}

int launch_ctr_bulk(const CtrArgs &a, int nr, const Shape &sh, hipStream_t st)
{
    const CtrKeys keys = ctr_keys(a);
    (void)hipGetLastError();   // not ours: left by earlier calls
    if (nr == 10)
        hipLaunchKernelGGL(ctr_bulk_kernel<10>, dim3(sh.grid), dim3(kBulkWG), 0, st, a.in, a.out, a.len, a.ctr0, a.x0,
                           keys);
    else if (nr == 14)
        hipLaunchKernelGGL(ctr_bulk_kernel<14>, dim3(sh.grid), dim3(kBulkWG), 0, st, a.in, a.out, a.len, a.ctr0, a.x0,
                           keys);
    else
        return AES_EINVAL;
    return launch_status();
}

}  // namespace aesctr
