// batch.cpp -- aes_ctr_crypt_batch: descriptor table staging and launch.
//
// Per (device, stream) the library keeps a context: a ring of slots, each a
// pinned host buffer for one launch's table (header + up to kMaxBatch
// descriptors, their inline keys and key installs) and the device table it is
// uploaded to.  A call fills a free slot and launches two kernels on the
// caller's stream: one that copies the slot into its table, then the batch
// kernel over it; with use_graph they are the two nodes of an executable HIP
// graph that the slot keeps, whose copy size is set before each launch (nothing
// is re-captured between calls).
//
// A slot, with its table and graph, is used again only after the event recorded
// behind its last launch has been waited for on the host.  Nothing else orders
// calls, so it does not matter which queue a stream handle stands for:
// hipStreamPerThread is one value and a stream of its own in every thread, and a
// new stream may get the address of a destroyed one whose work still runs.
//
// The tile counter the kernel claims work from is part of every upload (0), so
// no memset node is needed.  The call cannot itself be captured into a caller's
// graph (its staging would be rewritten by later calls): on a capturing stream
// it returns AES_EINVAL.
#include <algorithm>
#include <map>
#include <memory>
#include <mutex>
#include <string.h>
#include <vector>

#include "aesctr_internal.h"
#include "host_pool.h"
#include "tune.h"

namespace aesctr {

namespace {

constexpr int kSlots = 4;
constexpr size_t kTableBytes = (kMaxTableBytes + 15) & ~size_t(15);   // the upload moves whole quads
constexpr size_t kTableStride = (kTableBytes + 255) & ~size_t(255);

// Descriptors per part of the host's parallel validation.
constexpr size_t kCheckGrain = 4096;

struct BatchShape {
    int tile_bytes, wg, grid, bpl, use_graph;
};

struct SlotGraph {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipGraphNode_t upload_node = nullptr;
    int grid = 0, bpl = 0;
};

struct BatchCtx {
    std::mutex mu;
    int device = -1;
    void *dev_table[kSlots] = {};
    uint8_t *staging[kSlots] = {};
    const void *staging_view[kSlots] = {};   // the pinned slots' device addresses
    hipEvent_t done[kSlots] = {};
    bool used[kSlots] = {};
    SlotGraph g[kSlots];
    int next_slot = 0;
};

std::mutex g_ctx_mu;
// Contexts live until process exit (freeing them from a static destructor
// could run after the HIP runtime has shut down).  A stream's context goes
// back to its device's free list when the stream is retired
// (release_batch_stream, called by aes_engine_destroy before it destroys its
// streams), and the next new stream on that device takes it over, so
// creating and destroying engines does not grow memory.
std::map<std::pair<int, void *>, BatchCtx *> g_ctx;
std::map<int, std::vector<BatchCtx *>> g_free;

int init_ctx(BatchCtx *c, int device)
{
    c->device = device;
    // One allocation for all four: each in its own, 1000 requests of 1 KiB take 27.4
    // us a call (26.8), 4096 of them 55.4 (54.2).
    uint8_t *tables = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(&tables), kSlots * kTableStride) != hipSuccess)
        return AES_ENOMEM;
    for (int i = 0; i < kSlots; ++i) {
        // Coherent (fine-grained): the upload kernel reads the slot, and a
        // reused slot must never be served from a line cached by an earlier
        // launch.
        if (hipHostMalloc(reinterpret_cast<void **>(&c->staging[i]), kTableBytes, hipHostMallocCoherent) !=
            hipSuccess)
            return AES_ENOMEM;
        c->dev_table[i] = tables + i * kTableStride;
        void *view = nullptr;
        if (hipHostGetDevicePointer(&view, c->staging[i], 0) != hipSuccess || !view)
            return AES_EDEVICE;
        c->staging_view[i] = view;
        if (hipEventCreateWithFlags(&c->done[i], hipEventDisableTiming) != hipSuccess)
            return AES_EDEVICE;
    }
    return AES_OK;
}

BatchCtx *get_ctx(int device, void *stream, int *rc)
{
    std::lock_guard<std::mutex> lk(g_ctx_mu);
    auto key = std::make_pair(device, stream);
    auto it = g_ctx.find(key);
    if (it != g_ctx.end()) {
        *rc = AES_OK;
        return it->second;
    }
    std::vector<BatchCtx *> &fl = g_free[device];
    if (!fl.empty()) {
        BatchCtx *c = fl.back();
        fl.pop_back();
        g_ctx[key] = c;
        *rc = AES_OK;
        return c;
    }
    BatchCtx *c = new BatchCtx();
    *rc = init_ctx(c, device);
    if (*rc != AES_OK) {
        note_device_error(hipGetLastError());
        return nullptr;   // partially initialised context is leaked deliberately
    }
    g_ctx[key] = c;
    return c;
}

// Capture (upload of slot s into the table) + kernel on a private stream.
int build_graph(BatchCtx *c, int s, int grid, int bpl)
{
    SlotGraph &sg = c->g[s];
    if (sg.exec) {
        (void)hipGraphExecDestroy(sg.exec);
        (void)hipGraphDestroy(sg.graph);
        sg = SlotGraph{};
    }
    hipStream_t cap;
    if (hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess)
        return AES_EDEVICE;
    int rc = AES_OK;
    if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
        rc = AES_EDEVICE;
    } else {
        int lrc = launch_upload(c->staging_view[s], c->dev_table[s], kTableBytes / 16, cap);
        if (lrc == AES_OK)
            lrc = launch_ctr_batch(c->dev_table[s], grid, 1024, bpl, cap);
        hipGraph_t g = nullptr;
        if (hipStreamEndCapture(cap, &g) != hipSuccess || lrc != AES_OK || !g) {
            rc = lrc != AES_OK ? lrc : AES_EDEVICE;
        } else {
            sg.graph = g;
            size_t roots = 1;
            if (hipGraphGetRootNodes(g, &sg.upload_node, &roots) != hipSuccess || roots != 1)
                sg.upload_node = nullptr;
            if (!sg.upload_node || hipGraphInstantiate(&sg.exec, g, nullptr, nullptr, 0) != hipSuccess)
                rc = AES_EDEVICE;
        }
    }
    (void)hipStreamDestroy(cap);
    if (rc != AES_OK) {
        note_device_error(hipGetLastError());
        sg.exec = nullptr;
        return rc;
    }
    sg.grid = grid;
    sg.bpl = bpl;
    return AES_OK;
}

}  // namespace

uint32_t batch_own_tiles(uint64_t tiles, int grid)
{
    // A claim from the header's counter is a device-wide atomic on one word:
    // about 13 ns each, however many waves ask, and when every wave asks at
    // its first tile the queue is 50 us long.  So a launch of few tiles makes
    // none, and a large one leaves a twelfth to them, more than the CUs differ
    // by at the end of equal shares (3-6%).
    const uint64_t per_wg = (tiles + grid - 1) / grid;
    return static_cast<uint32_t>(per_wg >= 64 ? per_wg - per_wg / 12 : per_wg);
}

// Tiles of tile_blocks blocks from a request's start.
static uint64_t plain_tiles(uint64_t len, uint32_t tile_blocks)
{
    return len / (16 * tile_blocks) + (len % (16 * tile_blocks) != 0);
}

// Completes a staged table at buf: n descriptors, header.n_keys inline keys
// and header.n_install installs written.  Assigns first tiles and fills the
// rest of the header.  Returns the bytes to upload, or 0 if the tile count
// would overflow.
size_t finish_stage(uint8_t *buf, size_t n, uint32_t tile_blocks, int grid, bool plain)
{
    BatchHeader *h = reinterpret_cast<BatchHeader *>(buf);
    BatchDesc *out = reinterpret_cast<BatchDesc *>(buf + sizeof(BatchHeader));
    uint64_t tiles = 0;
    for (size_t i = 0; i < n; ++i) {
        out[i].tile0 = static_cast<uint32_t>(tiles);
        tiles += plain ? plain_tiles(out[i].len, tile_blocks) : request_tiles(out[i].len, out[i].ctr0, tile_blocks);
        if (tiles > 0x7fffffffu)
            return 0;
    }
    h->n = static_cast<uint32_t>(n);
    h->total_tiles = static_cast<uint32_t>(tiles);
    h->tile_blocks = tile_blocks;
    h->next = 0;
    h->own_tiles = batch_own_tiles(tiles, grid);
    h->keys_off = static_cast<uint32_t>(batch_keys_off(n));
    h->install_off = static_cast<uint32_t>(batch_install_off(n, h->n_keys));
    memset(h->pad, 0, sizeof(h->pad));
    return batch_table_bytes(n, h->n_keys, h->n_install);
}

namespace {

// Records per part of the host's parallel record building.
constexpr size_t kRecordGrain = 256;

// Whether the requests in a staged table run with four lanes per block
// (ctr_quad_table_kernel): at most two of its workgroups for each of `cus`, the
// small batch's limit, and no more requests than its waves look through.  us per
// call back to back, and for one call up to its end, in brackets as tiles of the
// table kernel: 9 requests of 0.1-1 KB 10.4 (15.0) and 18.2 (22.4), 64 of them 11.1
// (15.4) and 20.0 (24.3), 256 of 0.1-4 KB 14.6 (17.1) and 26.2 (29.7), 12 of 20-60
// KB 11.2 (15.3) and 19.4 (23.0).  Not through a captured graph, whose second node
// is the table kernel, nor where the caller names that kernel's tiles, blocks per
// lane or workgroup size.
bool quad_table(const BatchDesc *descs, size_t n, int cus)
{
    if (n > kQuadTableReqs)
        return false;
    uint64_t tiles = 0;
    for (size_t i = 0; i < n; ++i)
        tiles += plain_tiles(descs[i].len, kQuadTileBlocks);
    return tiles <= 2 * static_cast<uint64_t>(cus);
}

// How the tiles of a small batch are cut for `waves` waves (run_tile): by position,
// where a request whose first counter is ctr0 mod 64 != 0 (`odd`: one is) lies across
// the memory's lines and may need one step or tile more, or from its start, where
// every step takes 3 to 8% longer.
//  * One round of all waves takes as long as its longest tile, so an odd batch goes
//    from the start: 4 requests of 8 KiB in one tile each from counter 1 19.8 us by
//    position and 18.1 from the start, 4 of 300,000 bytes 8.7 and 8.5.
//  * More rounds: from the start where the further tiles make one more: one request
//    of 4 MiB from counter 1 (2049 or 2048 tiles, 2048 waves) 9.5 and 7.7, four of 1
//    MiB 11.4 and 9.3, eight of 8 MiB (two rounds) 74.0 and 67.9.  Not so among
//    thirteen rounds, four where tiles have over 256 blocks (eight requests of 32 MiB
//    246 and 259), nor for one or two such tiles, which a workgroup's oldest wave takes
//    while the others still work (one of 32 MiB 26.8 and 28.7, two of 16 MiB 31.9 and
//    33.8).
bool by_position(uint64_t plain, uint64_t shifted, bool odd, uint64_t waves, uint32_t tile_blocks)
{
    const uint64_t rounds = (plain + waves - 1) / waves;
    const bool large = tile_blocks > 256;
    if (rounds <= 1)
        return !odd;
    return (shifted + waves - 1) / waves == rounds || rounds >= (large ? 4 : 13) || (large && shifted - plain <= 2);
}

// A batch of at most kSmallBatch requests goes in the kernel's argument block
// (no staging slot, no upload), to one of three kernels whose grid it sizes.
// Where four lanes per block make at most two workgroups for each of `cus`, the
// requests run so (ctr_quad.hip); else with two lanes per block where that makes at
// most one (ctr_pair.hip); the limits are the single message's (quad_shape,
// pair_shape), and cus the smaller of the grid and the chip's CUs: beyond two
// workgroups per CU a wave per tile is faster (4 requests of 1 MiB 9.3 us against
// 11.7 as quads, of 4 MiB 23.8 against 36.6), which a larger grid does not change.
// Else a wave per tile in workgroups of four waves, at most two workgroups per
// workgroup of `grid`, the waves looping over further tiles.  us per call back to back, and for
// one call up to its end, in brackets those of the last kernel.  Quads: one
// request of 64 KiB 4.6 (7.8) and 15.2 (19.5); one of 512 KiB 4.6 (8.0) and 16.0
// (19.6); 8 of 100 bytes 4.8 (8.7) and 15.2 (19.3); 8 of 64 KiB 4.8 (9.6) and 16.0
// (21.4), in pinned host memory 30.2 (33.4) for one call.  Pairs: one request of 1
// MiB 4.8 (8.1) and 17.0 (20.2); 8 of 128 KiB 4.8 (9.6) and 16.9 (21.9), in pinned
// host memory 47.5 (49.7).
// several: whether the first two may take it (not where the caller names the last
// one's tiles or blocks per lane).  Returns AES_OK, AES_ERANGE or AES_EDEVICE.
int launch_small(hipStream_t st, const LaunchSpec &spec, uint32_t tile_blocks, int grid, int cus, int bpl, bool several)
{
    SmallBatchArgs args{};
    const uint64_t cap = 2 * static_cast<uint64_t>(grid), pair_cap = static_cast<uint64_t>(cus), quad_cap = 2 * pair_cap;
    uint64_t quads = 0, pairs = 0, plain = 0, shifted = 0;
    bool odd = false;
    for (size_t i = 0; i < spec.n; ++i) {
        const BatchDesc &d = spec.descs[i];
        quads += plain_tiles(d.len, kQuadTileBlocks);
        pairs += plain_tiles(d.len, kPairTileBlocks);
        plain += plain_tiles(d.len, tile_blocks);
        shifted += request_tiles(d.len, d.ctr0, tile_blocks);
        odd = odd || (d.len != 0 && (d.ctr0 & 63u) != 0);
    }
    const bool quad = several && quads <= quad_cap;
    const bool pair = several && !quad && pairs <= pair_cap;
    if (quad || pair)
        tile_blocks = quad ? kQuadTileBlocks : kPairTileBlocks;
    const bool shift = !quad && !pair && by_position(plain, shifted, odd, 4 * quad_cap, tile_blocks);
    uint64_t tiles = 0;
    for (size_t i = 0; i < spec.n; ++i) {
        const BatchDesc &d = spec.descs[i];
        SmallRec &r = args.r[i];
        r.in = d.in;
        r.out = d.out;
        r.len = d.len;
        r.ctr0 = d.ctr0;
        r.x0 = d.x0;
        r.nr = d.nr;
        memcpy(r.k1, d.k1, sizeof(r.k1));
        r.key = d.key;
        r.install = kNoInstall;
        if (!(d.key & kKeyResident)) {
            memcpy(r.rk, spec.keys[d.key].rk, sizeof(r.rk));
            for (size_t j = 0; j < spec.n_install; ++j)
                if (spec.installs[j].key == d.key)
                    r.install = spec.installs[j].slot;
        }
        r.tile0 = static_cast<uint32_t>(tiles);
        tiles += shift ? request_tiles(d.len, d.ctr0, tile_blocks) : plain_tiles(d.len, tile_blocks);
        if (tiles > 0x7fffffffu)
            return AES_ERANGE;
    }
    // An install names one inline key; two records sharing that key must not
    // both write the slot: keep the first.
    for (size_t i = 0; i < spec.n; ++i)
        for (size_t j = 0; j < i; ++j)
            if (args.r[i].install != kNoInstall && args.r[i].install == args.r[j].install)
                args.r[i].install = kNoInstall;
    args.n = static_cast<uint32_t>(spec.n);
    args.total_tiles = static_cast<uint32_t>(tiles);
    args.tile_blocks = tile_blocks;
    args.resident = spec.resident;
    if (quad)
        return launch_ctr_quad_batch(args, st);
    if (pair)
        return launch_ctr_pair_batch(args, st);
    const uint64_t want = (tiles + 3) / 4;
    const int small_grid = static_cast<int>(std::max<uint64_t>(1, std::min(want, cap)));
    return launch_ctr_batch_small(args, small_grid, bpl, shift, st);
}

// Takes the context's next staging slot once its last launch has finished.
int take_slot(BatchCtx *c, int *slot)
{
    *slot = c->next_slot;
    c->next_slot = (c->next_slot + 1) % kSlots;
    if (c->used[*slot] && hipEventSynchronize(c->done[*slot]) != hipSuccess) {
        note_device_error(hipGetLastError());
        return AES_EDEVICE;
    }
    return AES_OK;
}

// Uploads the first `bytes` of staging slot `slot` into its device table and
// launches the batch kernel on st, as two plain launches or through the slot's
// captured graph of them, then marks the slot busy until that work finishes.
int submit_slot(BatchCtx *c, int slot, size_t bytes, hipStream_t st, int grid, int bpl, bool use_graph, bool quad)
{
    int rc = AES_OK;
    void *table = c->dev_table[slot];
    const uint32_t quads = static_cast<uint32_t>((bytes + 15) / 16);
    if (use_graph) {
        SlotGraph &sg = c->g[slot];
        if (!sg.exec || sg.grid != grid || sg.bpl != bpl) {
            if ((rc = build_graph(c, slot, grid, bpl)) != AES_OK)
                return rc;
        }
        if (set_upload_node(sg.exec, sg.upload_node, c->staging_view[slot], table, quads) != hipSuccess ||
            hipGraphLaunch(sg.exec, st) != hipSuccess) {
            note_device_error(hipGetLastError());
            rc = AES_EDEVICE;
        }
    } else if ((rc = launch_upload(c->staging_view[slot], table, quads, st)) == AES_OK) {
        rc = quad ? launch_ctr_quad_table(table, *reinterpret_cast<const BatchHeader *>(c->staging[slot]), st)
                  : launch_ctr_batch(table, grid, 1024, bpl, st);
    }
    // Behind a launch that failed too: the upload ahead of it may be queued, and
    // the slot must not be rewritten before that has ended.
    if (hipEventRecord(c->done[slot], st) != hipSuccess) {
        note_device_error(hipGetLastError());
        (void)hipStreamSynchronize(st);
        return AES_EDEVICE;
    }
    c->used[slot] = true;
    return rc;
}

}  // namespace

int launch_spec(int device, hipStream_t st, const LaunchSpec &spec, int tile_bytes, int grid, int bpl,
                bool use_graph, bool allow_small)
{
    const uint32_t tile_blocks = static_cast<uint32_t>(tile_bytes / 16);
    if (spec.n == 0)
        return AES_OK;
    if (spec.n > static_cast<size_t>(kMaxBatch) || spec.n_keys > static_cast<size_t>(kMaxBatch) ||
        spec.n_install > static_cast<size_t>(kMaxBatch))
        return AES_EINVAL;
    if (allow_small && spec.n <= kSmallBatch)
        return launch_small(st, spec, tile_blocks, grid, grid, bpl, true);
    int rc;
    BatchCtx *c = get_ctx(device, st, &rc);
    if (!c)
        return rc;
    std::lock_guard<std::mutex> lk(c->mu);
    int slot;
    if ((rc = take_slot(c, &slot)) != AES_OK)
        return rc;
    uint8_t *buf = c->staging[slot];
    BatchHeader *h = reinterpret_cast<BatchHeader *>(buf);
    memset(h, 0, sizeof(*h));
    h->n_keys = static_cast<uint32_t>(spec.n_keys);
    h->n_install = static_cast<uint32_t>(spec.n_install);
    h->resident = spec.resident;
    memcpy(buf + sizeof(BatchHeader), spec.descs, spec.n * sizeof(BatchDesc));
    memcpy(buf + batch_keys_off(spec.n), spec.keys, spec.n_keys * sizeof(KeyRec));
    memcpy(buf + batch_install_off(spec.n, spec.n_keys), spec.installs, spec.n_install * sizeof(InstallRec));
    const bool quad = !use_graph && allow_small && quad_table(spec.descs, spec.n, grid);
    const size_t bytes = finish_stage(buf, spec.n, quad ? kQuadTileBlocks : tile_blocks, grid, quad);
    if (bytes == 0)
        return AES_ERANGE;
    return submit_slot(c, slot, bytes, st, grid, bpl, use_graph, quad);
}

void release_batch_stream(int device, hipStream_t st)
{
    BatchCtx *c = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_ctx_mu);
        auto it = g_ctx.find(std::make_pair(device, static_cast<void *>(st)));
        if (it == g_ctx.end())
            return;
        c = it->second;
        g_ctx.erase(it);
    }
    {
        // The stream's last launches read the staging slots: wait for them
        // before another stream may refill a slot.
        std::lock_guard<std::mutex> lk(c->mu);
        for (int i = 0; i < kSlots; ++i) {
            if (c->used[i] && hipEventSynchronize(c->done[i]) != hipSuccess)
                note_device_error(hipGetLastError());
            c->used[i] = false;
        }
    }
    std::lock_guard<std::mutex> lk(g_ctx_mu);
    g_free[device].push_back(c);
}

uint64_t batch_tile_bytes(uint64_t batch_bytes, int num_cus)
{
    // About kTilesPerCu tiles per CU (one per wave of a workgroup), between
    // 2 KiB (one wave step: 64 lanes x 2 blocks) and kMaxTile, multiples of
    // 2 KiB; the tune cache's batch entry may set both constants.  Measured on
    // MI355X: on the 4096-request workload 64 KiB tiles (3.59 ms) beat 16 KiB
    // (3.67) and 4 KiB (12.8, when every tile was claimed with an atomic);
    // small batches need small tiles to reach many CUs.
    constexpr uint64_t kTilesPerCu = 16, kMaxTile = 65536;
    uint64_t tpc = kTilesPerCu, max_tile = kMaxTile;
    TuneEntry te;
    if (tune_lookup_batch(&te)) {
        if (te.tiles_per_cu >= 1 && te.tiles_per_cu <= 1024)
            tpc = static_cast<uint64_t>(te.tiles_per_cu);
        if (te.max_tile_bytes >= 2048 && te.max_tile_bytes <= (1 << 24) && te.max_tile_bytes % 2048 == 0)
            max_tile = static_cast<uint64_t>(te.max_tile_bytes);
    }
    const uint64_t cus = static_cast<uint64_t>(num_cus > 0 ? num_cus : 1);
    uint64_t tile = (batch_bytes / (tpc * cus) + 2047) & ~uint64_t(2047);
    return tile < 2048 ? 2048 : tile > max_tile ? max_tile : tile;
}

int batch_blocks_per_lane()
{
    TuneEntry te;
    return tune_lookup_batch(&te) && (te.bpl == 1 || te.bpl == 2) ? te.bpl : 2;
}

// Descriptor (key field left 0) and round keys of one validated request.
void make_batch_desc(const aes_ctr_desc_t &d, BatchDesc *o, KeyRec *k)
{
    KeyMaterial km;
    make_key_material(*d.sched, d.nonce, &km);
    memset(o, 0, sizeof(*o));
    o->in = reinterpret_cast<uint64_t>(d.in);
    o->out = reinterpret_cast<uint64_t>(d.out);
    o->len = d.len;
    o->ctr0 = d.ctr0;
    o->x0 = km.x0;
    o->nr = static_cast<uint32_t>(km.nr);
    memcpy(o->k1, km.k1, sizeof(o->k1));
    memset(k, 0, sizeof(*k));
    memcpy(k->rk, km.rk, sizeof(km.rk));
}

void make_batch_record(const aes_ctr_desc_t &d, RequestRec *o)
{
    make_batch_desc(d, &o->d, &o->key);
}

int check_desc(const aes_ctr_desc_t &d)
{
    int rc = check_sched(d.sched);
    if (rc != AES_OK)
        return rc;
    if (d.flags != 0)
        return AES_EINVAL;
    return check_buffers(d.in, d.out, d.len);
}

}  // namespace aesctr

using namespace aesctr;

extern "C" int aes_ctr_crypt_batch_cfg(const aes_ctr_desc_t *desc, size_t n, const aes_batch_cfg_t *cfg,
                                       void *stream)
{
    if (n == 0)
        return AES_OK;
    if (!desc)
        return AES_EINVAL;
    // Validation and the payload total, over parts in parallel; the status of
    // the first failing descriptor wins, as in a serial scan.
    struct Scan {
        int rc;
        uint64_t bytes;
    };
    const size_t parts = HostPool::parts(n, kCheckGrain);
    Scan scan[HostPool::kMaxParts];
    HostPool::get().parallel_for(n, kCheckGrain, [&](size_t p, size_t b, size_t e) {
        Scan r{AES_OK, 0};
        for (size_t i = b; i < e && r.rc == AES_OK; ++i) {
            r.rc = check_desc(desc[i]);
            r.bytes += desc[i].len;
        }
        scan[p] = r;
    });
    uint64_t total_bytes = 0;
    for (size_t p = 0; p < parts; ++p) {
        if (scan[p].rc != AES_OK)
            return scan[p].rc;
        total_bytes += scan[p].bytes;
    }
    // Tile size 0 = sized to the batch (batch_tile_bytes); two blocks per
    // lane unless the tune cache says otherwise.  Two plain launches (upload,
    // kernel): replaying a graph of them, which paid while the upload was a copy
    // of the runtime's, costs more at every size.  us per call up to its end (and
    // back to back), graph against plain: 9 requests of 0.1-1 KB 38.0 (23.4) and
    // 22.4 (15.2), 64 of 4 KiB-1 MiB 42.8 (31.7) and 33.6 (24.6), 1000 of 4-64 KiB
    // 82.3 (55.0) and 68.0 (42.0), 4096 of them 230 (138) and 204 (131).
    BatchShape sh{0, 1024, 0, batch_blocks_per_lane(), 0};
    if (cfg) {
        if (cfg->tile_bytes < 0 || (cfg->tile_bytes && (cfg->tile_bytes % 1024 != 0 || cfg->tile_bytes > (1 << 26))))
            return AES_EINVAL;
        if (cfg->wg_size != 0 && cfg->wg_size != 1024)
            return AES_EINVAL;
        if (cfg->grid < 0 || cfg->grid > kMaxBatchGrid ||
            (cfg->blocks_per_lane != 0 && cfg->blocks_per_lane != 1 && cfg->blocks_per_lane != 2))
            return AES_EINVAL;
        if (cfg->tile_bytes) sh.tile_bytes = cfg->tile_bytes;
        if (cfg->grid) sh.grid = cfg->grid;
        if (cfg->blocks_per_lane) sh.bpl = cfg->blocks_per_lane;
        sh.use_graph = cfg->use_graph;
    }
    // Several lanes per block, whose workgroups have tiles of their own, only for
    // callers who leave the tiles to the library.
    const bool several = !cfg || (cfg->tile_bytes == 0 && cfg->blocks_per_lane == 0);
    DeviceInfo di;
    int rc = device_info(&di);
    if (rc != AES_OK)
        return rc;
    if (sh.grid == 0)
        sh.grid = di.num_cus;
    const int cus = std::min(sh.grid, di.num_cus);

    hipStream_t st = static_cast<hipStream_t>(stream);
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
        note_device_error(hipGetLastError());
        return AES_EDEVICE;
    }
    if (cs != hipStreamCaptureStatusNone)
        return AES_EINVAL;

    if (sh.tile_bytes == 0)
        sh.tile_bytes = static_cast<int>(batch_tile_bytes(total_bytes, di.num_cus));
    const uint32_t tile_blocks = static_cast<uint32_t>(sh.tile_bytes / 16);

    // At most kSmallBatch requests: records in the kernel arguments.
    if (n <= kSmallBatch) {
        BatchDesc descs[kSmallBatch];
        KeyRec keys[kSmallBatch];
        for (size_t i = 0; i < n; ++i) {
            make_batch_desc(desc[i], &descs[i], &keys[i]);
            descs[i].key = static_cast<uint32_t>(i);
        }
        LaunchSpec spec;
        spec.descs = descs;
        spec.n = n;
        spec.keys = keys;
        spec.n_keys = n;
        return launch_small(st, spec, tile_blocks, sh.grid, cus, sh.bpl, several);
    }

    // Otherwise launches of up to kMaxBatch requests, each request's key
    // inline.  Records are built straight into the pinned staging slot.
    BatchCtx *c = get_ctx(di.ordinal, st, &rc);
    if (!c)
        return rc;
    std::lock_guard<std::mutex> lk(c->mu);
    for (size_t first = 0; first < n; first += kMaxBatch) {
        const size_t m = n - first < static_cast<size_t>(kMaxBatch) ? n - first : kMaxBatch;
        int slot;
        if ((rc = take_slot(c, &slot)) != AES_OK)
            return rc;
        uint8_t *buf = c->staging[slot];
        BatchHeader *h = reinterpret_cast<BatchHeader *>(buf);
        memset(h, 0, sizeof(*h));
        h->n_keys = static_cast<uint32_t>(m);
        BatchDesc *out = reinterpret_cast<BatchDesc *>(buf + sizeof(BatchHeader));
        KeyRec *keys = reinterpret_cast<KeyRec *>(buf + batch_keys_off(m));
        HostPool::get().parallel_for(m, kRecordGrain, [&](size_t, size_t b, size_t e) {
            for (size_t i = b; i < e; ++i) {
                make_batch_desc(desc[first + i], out + i, keys + i);
                out[i].key = static_cast<uint32_t>(i);
            }
        });
        const bool quad = several && !(cfg && cfg->wg_size) && sh.use_graph == 0 && quad_table(out, m, cus);
        const size_t bytes = finish_stage(buf, m, quad ? kQuadTileBlocks : tile_blocks, sh.grid, quad);
        if (bytes == 0)
            return AES_ERANGE;
        if ((rc = submit_slot(c, slot, bytes, st, sh.grid, sh.bpl, sh.use_graph != 0, quad)) != AES_OK)
            return rc;
    }
    return AES_OK;
}

extern "C" int aes_ctr_crypt_batch(const aes_ctr_desc_t *desc, size_t n, void *stream)
{
    return aes_ctr_crypt_batch_cfg(desc, n, nullptr, stream);
}
