// ctr_batch.hip -- one persistent launch over a table of requests (gfx950).
//
// Each workgroup fills the bank-replicated T-tables into LDS once (the same
// round code as the single-buffer kernel, ttable_device.h), copies the
// requests' first-tile indices into LDS, then its waves take the workgroup's
// own tiles from a counter in LDS and, in a large batch, the last twelfth from
// a device counter.  A tile is tile_blocks
// consecutive 16-byte blocks of one request; the wave finds the request by a
// binary search over the tile indices in LDS and reads that request's key
// material, pointers and counter parameters with scalar loads (they are the
// same for the whole wave).  Requests of any size, key length (AES-128 and
// AES-256 mixed) and alignment share the launch; dynamic claiming balances
// the log-uniform size mix.
//
// Bound: 4.5 GB in 4096 requests takes 3.0-3.2 ms at 129.7 (AES-128) or 193.8 table
// lookups per block, counted: 30 of the 32 per clock and CU that the LDS's two clocks
// per instruction allow, at the 1.9-2.0 GHz the card holds under this load (2.4
// without the payload traffic).
#include <stddef.h>

#include "ttable_tile.h"

namespace aesctr {
namespace {

constexpr int kBatchWG = 1024;
constexpr int kBatchLayout = kLayout4x32;
// The argument-path kernel (at most kSmallBatch requests, mostly a tile or
// two per wave) keeps the single-buffer kernel's small-message shape: 256
// threads, two tables x 32 copies (half the fill).
constexpr int kSmallWG = 256;
constexpr int kSmallLayout = kLayout2x32;

// Round keys are read through the constant address space, so they load with
// scalar instructions even though workgroup 0 of the same launch writes
// other slots of the resident table (installs): no launch reads a slot that
// it, or any launch in flight, writes.
typedef __attribute__((address_space(4))) const uint32_t c_u32;

// Tile t of request R (a BatchDesc in the device table or a SmallRec in the
// kernel arguments; both wave-uniform, so their fields arrive by scalar
// loads) with round keys rk (wave-uniform, read from the launch's inline keys
// or from a slot of the resident key table): the request's key material and
// pointers, then the tile's blocks.
template <int LAYOUT, int BPL, bool SHIFTED, class Rec>
__device__ __forceinline__ void request_tile(const TTable<LAYOUT> &tt, const Rec &R, const uint32_t (&rk)[60],
                                             uint32_t t, uint32_t tile_blocks, uint32_t lane)
{
    CtrArgs a;
    a.in = reinterpret_cast<const uint8_t *>(R.in);
    a.out = reinterpret_cast<uint8_t *>(R.out);
    a.len = R.len;
    a.ctr0 = R.ctr0;
    a.x0 = R.x0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        a.k1[c] = R.k1[c];
    const uint32_t nr = R.nr;
    const uint32_t nrk = 4 * (nr + 1);
#pragma unroll
    for (int i = 0; i < 60; ++i)
        a.rk[i] = i < 44 || nrk > 44 ? rk[i] : 0;
    const uint64_t positions = (SHIFTED ? message_shift(a.ctr0) : 0) + ((a.len + 15) >> 4);
    const uint64_t p0 = static_cast<uint64_t>(t - R.tile0) * tile_blocks;
    const uint64_t p1 = p0 + tile_blocks < positions ? p0 + tile_blocks : positions;
    // rotr(rk, 8) of rounds 2..Nr-1 for the two-table fold (the four-table
    // layout reads none).
    uint32_t krot[60];
    if constexpr (LAYOUT != kLayout4x32) {
#pragma unroll
        for (int i = 8; i < 56; ++i) krot[i] = rotr8(a.rk[i]);
    }
    if (nr == 10)
        run_tile<10, LAYOUT, BPL, SHIFTED>(tt, a, krot, p0, p1, lane);
    else
        run_tile<14, LAYOUT, BPL, SHIFTED>(tt, a, krot, p0, p1, lane);
}

// Writes the round keys of key record `src` (64 words) into slot `slot` of
// the resident table, one word per thread of the workgroup, with vector
// stores.  No wave of this launch reads that slot (its requests read the
// inline copy), and no launch in flight reads it either: the host hands a
// slot out for installing only when nothing references it.
__device__ __forceinline__ void install_key(uint32_t *resident, uint32_t slot, const uint32_t *src, uint32_t word)
{
    resident[64u * slot + word] = src[word];
}

// table: the uploaded header, descriptors, inline keys and installs,
// read-only here (so request fields come in through the scalar cache);
// counter: the header's `next` word.  Besides the outputs the kernel writes
// only that counter and, in workgroup 0, the installs' resident slots.
template <int BPL>
__global__ __launch_bounds__(kBatchWG) void ctr_batch_kernel(const uint8_t *__restrict__ table,
                                                             uint32_t *__restrict__ counter)
{
    __shared__ uint32_t lds[kLdsWords];
    __shared__ uint32_t s_tile0[kMaxBatch];
    __shared__ uint32_t s_next;

    const BatchHeader *hdr = reinterpret_cast<const BatchHeader *>(table);
    const BatchDesc *desc = reinterpret_cast<const BatchDesc *>(table + sizeof(BatchHeader));
    const uint32_t n = hdr->n;
    const uint32_t total = hdr->total_tiles;
    const uint32_t tile_blocks = hdr->tile_blocks;
    const uint32_t *keys = reinterpret_cast<const uint32_t *>(table + hdr->keys_off);
    uint32_t *resident = reinterpret_cast<uint32_t *>(hdr->resident);

    uint32_t tv[kFillStores / kBatchWG];
    fill_read<kBatchLayout, kBatchWG>(tv);
    for (uint32_t i = threadIdx.x; i < n; i += kBatchWG)
        s_tile0[i] = desc[i].tile0;
    if (blockIdx.x == 0) {
        const InstallRec *inst = reinterpret_cast<const InstallRec *>(table + hdr->install_off);
        const uint32_t words = 64u * hdr->n_install;
        for (uint32_t i = threadIdx.x; i < words; i += kBatchWG) {
            const InstallRec r = inst[i >> 6];
            install_key(resident, r.slot, keys + 64u * r.key, i & 63u);
        }
    }
    fill_write<kBatchLayout, kBatchWG>(lds, tv);
    if (threadIdx.x == 0)
        s_next = kBatchWG / 64;    // the waves' first tiles are their own numbers
    __syncthreads();

    const uint32_t lane = threadIdx.x & 63;
    TTable<kBatchLayout> tt{reinterpret_cast<const char *>(lds), 4 * (lane & 31), 4 * (lane & 31) | 0x10000u};

    // Tile claiming.  Each workgroup owns hdr->own_tiles tiles, tile k * grid +
    // b being the k-th of workgroup b, and its waves take the next one from a
    // counter in LDS (older waves win the issue slots and finish first, so
    // equal shares per wave would leave the SIMDs to the youngest at the end).
    // What is left of a large batch after that is claimed from the header's
    // counter, one ahead of the tile in work: it evens out the CUs.  With a
    // claim from that counter by every wave at its first tile, 64 requests of
    // 12 MB in all took 50 us in this kernel; now 20.
    const uint32_t own = hdr->own_tiles, grid = gridDim.x;
    auto next_own = [&] {
        uint32_t k = 0;
        if (lane == 0)
            k = atomicAdd(&s_next, 1u);
        return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(k)));
    };
    auto claim = [&] {
        uint32_t k = 0;
        if (lane == 0)
            k = atomicAdd(counter, 1u);
        return k;
    };
    uint32_t k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t claimed = 0;
    for (bool mine = true;;) {
        uint32_t t;
        if (mine) {
            t = k * grid + blockIdx.x;
            if (k >= own) {
                mine = false;
                if (own * grid >= total)
                    break;
                claimed = claim();
            }
        }
        if (!mine) {
            t = own * grid + __builtin_amdgcn_readfirstlane(claimed);
            if (t < total)
                claimed = claim();
        }
        if (t >= total)
            break;
        // Last request whose first tile is <= t (empty requests share their
        // successor's tile0 and are skipped by taking the last match).
        uint32_t lo = 0, hi = n - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (s_tile0[mid] <= t)
                lo = mid;
            else
                hi = mid - 1;
        }
        const uint32_t r = __builtin_amdgcn_readfirstlane(lo);
        const BatchDesc &R = desc[r];
        const uint32_t key = R.key;
        uint32_t rk[60];
        if (key & kKeyResident) {
            c_u32 *p = (c_u32 *)(uintptr_t)(resident + 64u * (key & ~kKeyResident));
#pragma unroll
            for (int i = 0; i < 60; ++i) rk[i] = p[i];
        } else {
            const uint32_t *p = keys + 64u * key;
#pragma unroll
            for (int i = 0; i < 60; ++i) rk[i] = p[i];
        }
        request_tile<kBatchLayout, BPL, true>(tt, R, rk, t, tile_blocks, lane);
        if (mine)
            k = next_own();
    }
}

// The upload of a launch table from pinned staging: `quads` 16-byte pieces.  A
// kernel of the library's own because the copy that the runtime queues ahead of
// a launch costs more (64 requests, 20 KB of table: 33.4 -> 32.2 us a call; 9 of
// 4.5 MB 45.5 -> 43.5; an engine's first launch 7.6 -> 1.6 ms).  A table of 1.3 MB
// takes about 25 us either way, the rate of the PCIe link.
constexpr int kUploadWG = 256;
constexpr uint32_t kUploadGrid = 256;

__global__ __launch_bounds__(kUploadWG) void upload_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst,
                                                           uint32_t quads)
{
    for (uint32_t i = blockIdx.x * kUploadWG + threadIdx.x; i < quads; i += gridDim.x * kUploadWG)
        dst[i] = src[i];
}

// A batch of at most kSmallBatch requests whose records travel in the kernel
// argument block: no descriptor upload goes ahead of the launch (a separate
// host-to-device copy adds about 20 us to a small batch's latency).  Tiles
// are assigned statically, wave w taking tiles w, w + W, w + 2W, ... (W
// waves, numbered as in ctr_batch_kernel), so no work counter is needed.
// SHIFTED: how tiles are cut (see run_tile and launch_small).
template <int BPL, bool SHIFTED>
__global__ __launch_bounds__(kSmallWG) void ctr_batch_small_kernel(const SmallBatchArgs args)
{
    __shared__ uint32_t lds[layout_lds_words(kSmallLayout)];

    uint32_t tv[kFillStores / kSmallWG];
    fill_read<kSmallLayout, kSmallWG>(tv);
    uint32_t *resident = reinterpret_cast<uint32_t *>(args.resident);
    const uint32_t n = args.n;
    if (blockIdx.x == 0) {
        for (uint32_t j = threadIdx.x; j < 64u * n; j += kSmallWG) {
            const uint32_t i = j >> 6, w = j & 63u;
            if (args.r[i].install != kNoInstall && w < 60u)
                install_key(resident, args.r[i].install, args.r[i].rk, w);
        }
    }
    fill_write<kSmallLayout, kSmallWG>(lds, tv);
    __syncthreads();

    const uint32_t lane = threadIdx.x & 63;
    TTable<kSmallLayout> tt{reinterpret_cast<const char *>(lds), 4 * (lane & 31), 4 * (lane & 31) | 0x10000u};
    const uint32_t waves = gridDim.x * (kSmallWG / 64);
    for (uint32_t t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * gridDim.x + blockIdx.x;
         t < args.total_tiles; t += waves) {
        // Last request whose first tile is <= t (skips empty requests).
        uint32_t r = 0;
        for (uint32_t i = 1; i < n; ++i)
            if (args.r[i].tile0 <= t)
                r = i;
        const SmallRec &R = args.r[r];
        uint32_t rk[60];
        if (R.key & kKeyResident) {
            c_u32 *p = (c_u32 *)(uintptr_t)(resident + 64u * (R.key & ~kKeyResident));
#pragma unroll
            for (int i = 0; i < 60; ++i) rk[i] = p[i];
        } else {
#pragma unroll
            for (int i = 0; i < 60; ++i) rk[i] = R.rk[i];
        }
        request_tile<kSmallLayout, BPL, SHIFTED>(tt, R, rk, t, args.tile_blocks, lane);
    }
}

}  // namespace

namespace {

uint32_t upload_grid(uint32_t quads)
{
    const uint32_t g = (quads + kUploadWG - 1) / kUploadWG;
    return g < 1 ? 1 : g > kUploadGrid ? kUploadGrid : g;
}

}  // namespace

int launch_upload(const void *src, void *dst, uint32_t quads, hipStream_t st)
{
    (void)hipGetLastError();   // not ours: left by earlier calls
    hipLaunchKernelGGL(upload_kernel, dim3(upload_grid(quads)), dim3(kUploadWG), 0, st, static_cast<const u32x4 *>(src),
                       static_cast<u32x4 *>(dst), quads);
    return launch_status();
}

hipError_t set_upload_node(hipGraphExec_t exec, hipGraphNode_t node, const void *src, void *dst, uint32_t quads)
{
    void *args[3] = {&src, &dst, &quads};
    hipKernelNodeParams kp{};
    kp.func = reinterpret_cast<void *>(upload_kernel);
    kp.gridDim = dim3(upload_grid(quads));
    kp.blockDim = dim3(kUploadWG);
    kp.kernelParams = args;
    return hipGraphExecKernelNodeSetParams(exec, node, &kp);
}

int launch_ctr_batch(const void *dev_table, int grid, int wg, int bpl, hipStream_t st)
{
    if (wg != kBatchWG || grid <= 0 || grid > kMaxBatchGrid)
        return AES_EINVAL;
    const uint8_t *t = static_cast<const uint8_t *>(dev_table);
    uint32_t *ctr = reinterpret_cast<uint32_t *>(const_cast<uint8_t *>(t) + offsetof(BatchHeader, next));
    (void)hipGetLastError();   // not ours: left by earlier calls
    switch (bpl) {
    case 1: hipLaunchKernelGGL(ctr_batch_kernel<1>, dim3(grid), dim3(kBatchWG), 0, st, t, ctr); break;
    case 2: hipLaunchKernelGGL(ctr_batch_kernel<2>, dim3(grid), dim3(kBatchWG), 0, st, t, ctr); break;
    default: return AES_EINVAL;
    }
    return launch_status();
}

int launch_ctr_batch_small(const SmallBatchArgs &args, int grid, int bpl, bool shifted, hipStream_t st)
{
    if (grid <= 0 || grid > kMaxBatchGrid || args.n > kSmallBatch || (bpl != 1 && bpl != 2))
        return AES_EINVAL;
    (void)hipGetLastError();   // not ours: left by earlier calls
    auto kernel = shifted ? (bpl == 1 ? ctr_batch_small_kernel<1, true> : ctr_batch_small_kernel<2, true>)
                          : (bpl == 1 ? ctr_batch_small_kernel<1, false> : ctr_batch_small_kernel<2, false>);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSmallWG), 0, st, args);
    return launch_status();
}

}  // namespace aesctr
