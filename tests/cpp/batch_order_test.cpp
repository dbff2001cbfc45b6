// Order of a batch call's device work against the calls before it, in a model of
// HIP's queues.  The library keeps its device tables by stream handle, but a
// handle may stand for several queues (hipStreamPerThread is one value in every
// thread; a destroyed stream's address comes back), and a launch may fail after
// the table's upload is queued.  Every upload has to be ordered behind all work
// that reads or writes the table, and a pinned slot is rewritten only when the
// upload from it has ended.
//
// "routes" instead reads batches "requests bytes ctr0 tile_bytes blocks_per_lane
// grid use_graph" from stdin and prints the launch of each: "kernel tiles
// tile_blocks workgroups blocks_per_lane".
#include <stdio.h>
#include <stdlib.h>

#include <set>
#include <vector>

#include "aesctr_internal.h"

namespace {

struct Op {
    const void *table, *src;    // src: the pinned slot it reads, for uploads
    std::set<int> before;       // operations that have ended when it starts
};
struct Event {
    std::set<int> behind;
};
struct Graph {
    const void *src = nullptr, *table = nullptr;
};

std::vector<Op> g_ops;
std::set<int> g_tail[4];        // per queue: what its next operation waits for
std::set<int> g_host;           // operations the host has waited for
int g_queue = 0;                // the queue that stream handles stand for now
bool g_capturing = false, g_fail_kernel = false, g_routes = false;
Graph g_captured;
int g_races = 0;

void enqueue(const void *table, const void *src)
{
    Op op{table, src, g_tail[g_queue]};
    op.before.insert(g_host.begin(), g_host.end());
    for (size_t i = 0; i < g_ops.size(); ++i) {
        const int id = static_cast<int>(i);
        if (src && g_ops[i].table == table && !op.before.count(id)) {
            printf("upload %zu is not ordered behind operation %zu on its table\n", g_ops.size(), i);
            ++g_races;
        }
        if (src && g_ops[i].src == src && !g_host.count(id)) {
            printf("operation %zu reads a slot that upload %zu rewrote\n", i, g_ops.size());
            ++g_races;
        }
    }
    g_ops.push_back(op);
    op.before.insert(static_cast<int>(g_ops.size()) - 1);
    g_tail[g_queue] = op.before;
}

}  // namespace

hipError_t hipMalloc(void **p, size_t bytes) { return *p = calloc(1, bytes), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { return *p = calloc(1, bytes), hipSuccess; }
hipError_t hipHostGetDevicePointer(void **dev, void *host, unsigned) { return *dev = host, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = new Event, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    return static_cast<Event *>(e)->behind = g_tail[g_queue], hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    const Event &ev = *static_cast<Event *>(e);
    return g_host.insert(ev.behind.begin(), ev.behind.end()), hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned)
{
    const Event &ev = *static_cast<Event *>(e);
    return g_tail[g_queue].insert(ev.behind.begin(), ev.behind.end()), hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    return g_host.insert(g_tail[g_queue].begin(), g_tail[g_queue].end()), hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned) { return *st = &g_captured, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    return *s = hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return g_capturing = true, hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    g_capturing = false;
    return *g = new Graph(g_captured), hipSuccess;
}
hipError_t hipGraphGetRootNodes(hipGraph_t g, hipGraphNode_t *nodes, size_t *n)
{
    return *nodes = g, *n = 1, hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    return *x = g, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    const Graph &g = *static_cast<Graph *>(x);
    enqueue(g.table, g.src);
    enqueue(g.table, nullptr);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }

namespace aesctr {

int launch_upload(const void *src, void *dst, uint32_t, hipStream_t)
{
    if (g_capturing)
        g_captured = Graph{src, dst};
    else
        enqueue(dst, src);
    return AES_OK;
}
hipError_t set_upload_node(hipGraphExec_t x, hipGraphNode_t, const void *src, void *dst, uint32_t)
{
    return *static_cast<Graph *>(x) = Graph{src, dst}, hipSuccess;
}
static int kernel(const char *name, const void *table, int grid, int bpl)
{
    if (g_fail_kernel)
        return AES_EDEVICE;
    if (g_capturing)
        return AES_OK;
    enqueue(table, nullptr);
    // The upload has not run: the table as staged.
    const BatchHeader *h = reinterpret_cast<const BatchHeader *>(g_ops[g_ops.size() - 2].src);
    if (g_routes)
        printf("%s %u %u %d %d\n", name, h->total_tiles, h->tile_blocks, grid, bpl);
    return AES_OK;
}
static int small(const char *name, const SmallBatchArgs &a, int grid, int bpl)
{
    if (g_routes)
        printf("%s %u %u %d %d\n", name, a.total_tiles, a.tile_blocks, grid, bpl);
    return AES_OK;
}
int launch_ctr_batch(const void *table, int grid, int, int bpl, hipStream_t) { return kernel("table", table, grid, bpl); }
int launch_ctr_quad_table(const void *table, const BatchHeader &h, hipStream_t)
{
    return kernel("quad_table", table, static_cast<int>(h.total_tiles), 0);
}
int launch_ctr_batch_small(const SmallBatchArgs &a, int grid, int bpl, bool shifted, hipStream_t)
{
    return small(shifted ? "small" : "small_plain", a, grid, bpl);
}
int launch_ctr_quad_batch(const SmallBatchArgs &a, hipStream_t) { return small("quad", a, a.total_tiles, 0); }
int launch_ctr_pair_batch(const SmallBatchArgs &a, hipStream_t) { return small("pair", a, a.total_tiles, 0); }
void note_device_error(hipError_t) {}
int device_info(DeviceInfo *out) { return *out = DeviceInfo{0, 256, 163840}, AES_OK; }
int check_sched(const aes_sched_t *) { return AES_OK; }
int check_buffers(const void *, const void *, uint64_t) { return AES_OK; }

}  // namespace aesctr

static int routes(const aes_sched_t &s)
{
    g_routes = true;
    unsigned long long n, len;
    unsigned ctr0;
    aes_batch_cfg_t cfg{};
    while (scanf("%llu %llu %u %d %d %d %d", &n, &len, &ctr0, &cfg.tile_bytes, &cfg.blocks_per_lane, &cfg.grid,
                 &cfg.use_graph) == 7) {
        std::vector<aes_ctr_desc_t> d(n);
        for (aes_ctr_desc_t &r : d) {
            r = aes_ctr_desc_t{};
            r.in = r.out = reinterpret_cast<void *>(uintptr_t(1) << 40);
            r.len = len;
            r.ctr0 = ctr0;
            r.sched = &s;
        }
        if (aes_ctr_crypt_batch_cfg(d.data(), d.size(), &cfg, nullptr) != AES_OK)
            return 1;
        if (cfg.use_graph && n > 8)
            printf("graph 0 0 0 0\n");
    }
    return 0;
}

int main(int argc, char **argv)
{
    const bool fail = argc > 1 && argv[1][0] == 'f';    // "failures", "handles" or "routes"
    const uint8_t key[16] = {};
    aes_sched_t s;
    if (aes_expand_key(key, 128, &s) != AES_OK)
        return 1;
    if (argc > 1 && argv[1][0] == 'r')
        return routes(s);
    uintptr_t handle = 2;    // a context of its own per scenario
    for (int use_graph = 0; use_graph < (fail ? 1 : 2); ++use_graph)    // (a failed graph launch queues nothing)
        for (uint64_t len : {uint64_t(100), uint64_t(1) << 20}) {
            std::vector<aes_ctr_desc_t> d(9);
            for (aes_ctr_desc_t &r : d) {
                r = aes_ctr_desc_t{};
                r.in = r.out = reinterpret_cast<void *>(uintptr_t(1) << 40);
                r.len = len;
                r.sched = &s;
            }
            aes_batch_cfg_t cfg{};
            cfg.use_graph = use_graph;
            hipStream_t st = reinterpret_cast<hipStream_t>(handle++);
            const int before = g_races;
            for (int call = 0; call < 14; ++call) {
                g_queue = call < 6 ? call & 1 : call == 6 ? 2 : 3;
                g_fail_kernel = fail && (call == 2 || call == 5 || call == 9);
                const int rc = aes_ctr_crypt_batch_cfg(d.data(), d.size(), &cfg, st);
                if (rc != (g_fail_kernel ? AES_EDEVICE : AES_OK))
                    return printf("call %d returned %d\n", call, rc), 1;
            }
            if (g_races != before)
                printf("graph %d, %llu bytes: races\n", use_graph, static_cast<unsigned long long>(len));
        }
    if (g_races)
        return 1;
    printf("batch order ok\n");
    return 0;
}
