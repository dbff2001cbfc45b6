// api.cpp -- C ABI entry points for single buffers: validation, launch-shape
// resolution and dispatch to the keystream kernels.
#include <mutex>
#include <string.h>

#include "aesctr_internal.h"
#include "tune.h"

namespace aesctr {

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_dev_mu;
DeviceInfo g_dev[kMaxDevices];
bool g_dev_ok[kMaxDevices];
thread_local hipError_t t_last_device_error = hipSuccess;

}  // namespace

void note_device_error(hipError_t e)
{
    if (e != hipSuccess)
        t_last_device_error = e;
}

int device_error()
{
    note_device_error(hipGetLastError());
    return AES_EDEVICE;
}

int launch_status()
{
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        return AES_OK;
    t_last_device_error = e;
    return AES_EDEVICE;
}

int device_info(DeviceInfo *out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        note_device_error(hipGetLastError());
        return AES_EDEVICE;
    }
    std::lock_guard<std::mutex> lk(g_dev_mu);
    if (!g_dev_ok[dev]) {
        DeviceInfo d{};
        d.ordinal = dev;
        if (hipDeviceGetAttribute(&d.num_cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipDeviceGetAttribute(&d.max_lds_per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
                hipSuccess) {
            note_device_error(hipGetLastError());
            return AES_EDEVICE;
        }
        g_dev[dev] = d;
        g_dev_ok[dev] = true;
    }
    *out = g_dev[dev];
    return AES_OK;
}

int check_sched(const aes_sched_t *s)
{
    if (!s)
        return AES_EINVAL;
    if (!((s->key_bits == 128 && s->nr == 10) || (s->key_bits == 256 && s->nr == 14)))
        return AES_EINVAL;
    return AES_OK;
}

// Argument checks shared by every entry point that takes a buffer pair.
int check_buffers(const void *in, const void *out, uint64_t len)
{
    if (len == 0)
        return AES_OK;
    if (!in || !out)
        return AES_EINVAL;
    if (len > (static_cast<uint64_t>(1) << 36))
        return AES_ERANGE;
    const uintptr_t a = reinterpret_cast<uintptr_t>(in);
    const uintptr_t b = reinterpret_cast<uintptr_t>(out);
    if (a > UINTPTR_MAX - len || b > UINTPTR_MAX - len)
        return AES_EINVAL;
    if (a != b && a < b + len && b < a + len)
        return AES_EOVERLAP;
    return AES_OK;
}

namespace {

// Whether a tuned T-table entry speaks for a message of this many blocks: its
// grid takes it in as many chunks as it took the size it was timed at.  Above
// that another shape may be better by a whole chunk (1.1 MiB in the shape tuned
// at 1 MiB: 5.00 us, in the rule's 3.65).
bool tuned_for(const TuneEntry &te, uint64_t blocks, uint64_t cus)
{
    const uint64_t pass = static_cast<uint64_t>(te.wg) * te.bpl * te.grid_per_cu * cus;
    const uint64_t tuned = ((uint64_t(1) << te.size_log2) + 15) / 16;
    return (blocks + pass - 1) / pass <= (tuned + pass - 1) / pass;
}

void take_entry(const TuneEntry &te, int num_cus, Shape *sh)
{
    sh->bpl = te.bpl;
    sh->wg = te.wg;
    sh->copies = te.copies;
    sh->tables = te.tables ? te.tables : (te.copies == 64 ? 2 : 4);
    sh->grid = te.grid_per_cu * num_cus;
    if (te.first >= kFirstWave0 && te.first <= kFirstFull &&
        first_chunk_mode_ok(te.first, sh->copies, sh->tables, sh->bpl, sh->wg))
        sh->wave_groups = te.first;
}

// The shape that a caller's explicit fields change where they name another than the
// default: one of the T-table kernel's
// own (ctr_ttable.hip), which every combination of them was built for.  The
// default's shapes above 16 MiB belong to another kernel (four tables, 1024
// threads): on top of those a mode or a block count alone would name a shape
// that does not exist, and 256 threads would run one small workgroup per CU
// (64 MiB in 86 us; from this base 49).
Shape explicit_base(int key_bits, uint64_t len, const DeviceInfo &di)
{
    Shape sh{};
    sh.variant = AES_VARIANT_TTABLE;
    sh.wave_groups = -1;
    TuneEntry te;
    if (tune_lookup(sh.variant, key_bits, len, &te)) {
        take_entry(te, di.num_cus, &sh);
        if (sh.wg == 1024 && sh.bpl == 2 && sh.tables == 4 && sh.wave_groups == kFirstWave0) {
            // An entry for the large-message kernel: the T-table kernel's best there.
            sh.wg = key_bits == 256 ? 1024 : 512;
            sh.bpl = key_bits == 256 ? 1 : 4;
            sh.tables = 2;
            sh.grid = 4 * di.num_cus;
        }
        return sh;
    }
    sh.grid = di.num_cus;
    sh.copies = 32;
    sh.tables = 2;
    const uint64_t per_cu = (len / 16) / static_cast<uint64_t>(di.num_cus > 0 ? di.num_cus : 1);
    if (per_cu >= 2048) {
        sh.bpl = per_cu >= 4096 ? 4 : 2;
        sh.wg = 512;
        sh.grid = 4 * di.num_cus;
    } else {
        sh.bpl = per_cu >= 1024 ? 2 : 1;
        sh.wg = per_cu >= 512 ? 512 : 256;
        sh.wave_groups = kFirstFull;
    }
    return sh;
}

// Whether a message of 16 to 32 MiB on 256 CUs runs in steps of a chunk per CU
// rather than in shared tiles, whose time grows with the length: where the last
// step is nearly full.  At 23 MiB, steps against tiles, AES-128 and AES-256: 17.9
// us against 18.6 and 23.7 against 25.0; with a partial block, which one thread
// takes behind its chunk, 18.8 against 18.7 and 24.1 against 25.1; at an odd
// address, where a wave's 1 KiB of payload touches one line more, 20.1 against 18.9
// and 25.0 against 24.9.  Third steps: from three quarters (AES-256: two thirds, 21.5
// MiB, 23.3 against 22.9).  Fourth steps: a full one (32 MiB 23.5 against 23.5);
// below that the tiles (31.5 MiB 23.4 against 23.4, with a partial block 24.2 against
// 23.5).
bool steps_fit(uint64_t len, uint64_t chunks, uint64_t cus, int key_bits, bool aligned)
{
    const uint64_t done = (chunks - 1) / cus, last = chunks - done * cus;
    if (done != 2)
        return done < 2 || last == cus;
    return aligned && (key_bits == 256 ? 3 * last >= 2 * cus : len % 16 == 0 && 4 * last >= 3 * cus);
}

// Whether cfg names any part of the launch shape.
bool names_shape(const aes_launch_cfg_t *cfg)
{
    return cfg && (cfg->blocks_per_lane || cfg->wg_size || cfg->grid || cfg->lds_copies || cfg->lds_tables ||
                   cfg->wave_groups);
}

// Whether cfg names a part of the launch shape that is not def's.
bool other_shape(const aes_launch_cfg_t &cfg, const Shape &def)
{
    auto other = [](int32_t field, int have) { return field != 0 && field != have; };
    return other(cfg.blocks_per_lane, def.bpl) || other(cfg.wg_size, def.wg) || other(cfg.grid, def.grid) ||
           other(cfg.lds_copies, def.copies) || other(cfg.lds_tables, def.tables) ||
           other(cfg.wave_groups, def.wave_groups == kFirstWave0 ? 3 : def.wave_groups);
}

}  // namespace

Shape default_shape(int variant, int key_bits, uint64_t len, bool aligned, const DeviceInfo &di)
{
    Shape sh{};
    sh.variant = variant == AES_VARIANT_AUTO ? AES_VARIANT_TTABLE : variant;
    sh.wave_groups = -1;    // first-chunk mode: the rule's (resolve_shape)
    TuneEntry te;
    const uint64_t cus = static_cast<uint64_t>(di.num_cus > 0 ? di.num_cus : 1);
    const uint64_t blocks = (len + 15) / 16;
    if (tune_lookup(sh.variant, key_bits, len, &te) &&
        (sh.variant != AES_VARIANT_TTABLE || tuned_for(te, blocks, cus))) {
        take_entry(te, di.num_cus, &sh);
    } else if (sh.variant == AES_VARIANT_TTABLE) {
        // The LDS holds only T0 and T2 (32 copies, 64 KiB): half the table
        // fill of four tables, for about 15% more VALU work per block, and
        // room for two workgroups per CU, so one workgroup's fill and
        // barriers overlap the other's keystream.  Time goes in steps: a
        // workgroup's chunk (workgroup size x blocks per lane) takes as long
        // full or nearly empty, so the shape is the one whose chunks fill the
        // CUs best, in blocks per CU.  us per launch at the ends of each range
        // (AES-128; in brackets the neighbouring shape there):
        //   up to 256   256 threads x 1 block, run as four lanes per block up to 128
        //               (ctr_quad.hip) and as two above (ctr_pair.hip):
        //                                    4 KiB 1.9, 512 KiB 2.4, 1 MiB 2.8
        //   up to 512   512 x 1              1.1 MiB 3.65 (5.00), 2 MiB 3.62 (5.21)
        //   up to 1024  512 x 2              2.2 MiB 5.07 (5.52), 4 MiB 5.17 (6.24)
        //   up to 1536  512 x 1, two per CU  4.3 MiB 6.42 (8.30), 6 MiB 6.42 (7.36)
        //   up to 2048  512 x 2, two per CU  6.8 MiB 7.57 (8.23), 8 MiB 7.65 (8.14)
        //   up to 2560  512 x 1, two per CU  8.2 MiB 8.71 (9.29), 9.8 MiB 9.10 (9.51)
        //   below 4096  512 x 2, two per CU  11.7 MiB 9.77 (10.48); four per CU: 13.7
        //                                    MiB 12.4 (12.7), 16 MiB 12.9 (13.1)
        // and 512 x 4, four per CU, from 16 MiB.  AES-256 has the same order.
        // Where every workgroup has one chunk (up to 1024), and with one block
        // per lane, rounds 1-2 of the first chunk run in full (first-chunk mode
        // 2: no group constants, no second barrier).
        // From 16 MiB on that shape takes steps of a chunk per CU (32 KiB x CUs), so it
        // stays only up to 32 MiB and where its last step is nearly full (steps_fit);
        // else one persistent workgroup per CU (ctr_bulk.hip), whose waves share 4 KiB
        // tiles.  AES-128: 16 MiB 13.0 us (bulk 13.4), 16 MiB + 100 bytes 17.0 (13.6),
        // 22 MiB 18.0 (17.7), 23 MiB 18.2 (18.5), 24 MiB 18.4 (19.0), 25 MiB 21.8
        // (19.9), 32 MiB 23.5 (23.5), 48 MiB 35.2 (31.1), 96.3 MiB 70.6 (60.4), 256 MiB
        // 167 (153); AES-256: 16 MiB 17.1 (17.7), 21 MiB 23.3 (22.6), 22 MiB 23.4 (24.1),
        // 24 MiB 24.3 (25.4), 32 MiB 31.0 (31.1), 48 MiB 47.6 (42.7), 256 MiB 230 (208).
        sh.grid = di.num_cus;
        sh.copies = 32;
        sh.tables = 2;
        sh.wg = 512;
        const uint64_t per_cu = (blocks + cus - 1) / cus;
        const uint64_t chunks = (blocks + 2047) / 2048;    // of 512 threads x 4 blocks
        if (per_cu <= 1024) {
            sh.bpl = per_cu > 512 ? 2 : 1;
            sh.wg = per_cu > 256 ? 512 : 256;
            sh.wave_groups = kFirstFull;
        } else if (per_cu <= 1536 || (per_cu > 2048 && per_cu <= 2560)) {
            sh.bpl = 1;
            sh.grid = 2 * di.num_cus;
            sh.wave_groups = kFirstFull;
        } else if (per_cu < 4096) {
            sh.bpl = 2;
            sh.grid = 2 * di.num_cus;
            sh.wave_groups = kFirstPerWave;
        } else if (per_cu <= 8192 && steps_fit(len, chunks, cus, key_bits, aligned)) {
            sh.bpl = 4;
            sh.grid = 4 * di.num_cus;
        } else {
            sh.bpl = 2;
            sh.wg = 1024;
            sh.tables = 4;
            sh.wave_groups = kFirstWave0;
        }
    } else if (sh.variant == AES_VARIANT_BITSLICE) {
        sh.bpl = 1;
        sh.wg = 256;
        sh.copies = 0;
        sh.tables = 0;
        sh.grid = 2 * di.num_cus;
    } else {
        // Vector-permute kernel: one block per lane, bound by VALU issue;
        // eight waves per CU keep every SIMD busy.
        sh.bpl = 1;
        sh.wg = 256;
        sh.copies = 0;
        sh.tables = 0;
        sh.grid = 2 * di.num_cus;
    }
    return sh;
}

// Never launch more workgroups than there is work for.
static void clamp_grid(Shape *sh, uint64_t len)
{
    uint64_t blocks = (len + 15) / 16;
    uint64_t per_wg;
    if (sh->variant == AES_VARIANT_BITSLICE)
        per_wg = static_cast<uint64_t>(sh->wg) * 8;    // 512 blocks per wave
    else
        per_wg = static_cast<uint64_t>(sh->wg) * sh->bpl;
    uint64_t need = (blocks + per_wg - 1) / per_wg;
    if (need < 1)
        need = 1;
    if (static_cast<uint64_t>(sh->grid) > need)
        sh->grid = static_cast<int>(need);
}

}  // namespace aesctr

using namespace aesctr;

extern "C" const char *aes_last_device_error(void)
{
    return hipGetErrorName(t_last_device_error);
}

extern "C" const char *aes_strerror(int status)
{
    switch (status) {
    case AES_OK: return "AES_OK: success";
    case AES_EINVAL: return "AES_EINVAL: invalid argument";
    case AES_ENOMEM: return "AES_ENOMEM: out of memory";
    case AES_EAGAIN: return "AES_EAGAIN: over the engine memory budget";
    case AES_ERANGE: return "AES_ERANGE: message longer than 2^32 blocks";
    case AES_EDEVICE: return "AES_EDEVICE: HIP device error or no device";
    case AES_ENOTFOUND: return "AES_ENOTFOUND: unknown ticket";
    case AES_ETIMEDOUT: return "AES_ETIMEDOUT: timed out";
    case AES_EOVERLAP: return "AES_EOVERLAP: input and output partially overlap";
    case AES_ECLOSED: return "AES_ECLOSED: engine is shutting down";
    case AES_ECANCELED: return "AES_ECANCELED: request canceled";
    case AES_ETOOBIG: return "AES_ETOOBIG: more requests than the fixed table holds";
    default: return "unknown aes status";
    }
}

namespace {

int check_cfg(const aes_launch_cfg_t *cfg, int *variant)
{
    *variant = cfg ? cfg->variant : AES_VARIANT_AUTO;
    if (*variant < AES_VARIANT_AUTO || *variant > AES_VARIANT_VPERM)
        return AES_EINVAL;
    if (cfg) {
        if (cfg->blocks_per_lane != 0 && cfg->blocks_per_lane != 1 && cfg->blocks_per_lane != 2 &&
            cfg->blocks_per_lane != 4)
            return AES_EINVAL;
        if (cfg->wg_size != 0 && (cfg->wg_size < 64 || cfg->wg_size > 1024 || cfg->wg_size % 64 != 0))
            return AES_EINVAL;
        if (cfg->grid < 0 || (cfg->lds_copies != 0 && cfg->lds_copies != 32 && cfg->lds_copies != 64))
            return AES_EINVAL;
        if (cfg->lds_tables != 0 && cfg->lds_tables != 2 && cfg->lds_tables != 4)
            return AES_EINVAL;
        if (cfg->lds_copies == 64 && cfg->lds_tables == 4)   // 256 KiB: more than a CU's LDS
            return AES_EINVAL;
        if (cfg->wave_groups < 0 || cfg->wave_groups > 3)
            return AES_EINVAL;
    }
    return AES_OK;
}

// The launch shape for len bytes: the default (or tuned) shape, overridden
// by the non-zero fields of cfg, with the grid clamped to the work.  aligned: in
// and out are at multiples of 16 bytes.
Shape resolve_shape(int variant, int key_bits, uint64_t len, bool aligned, const aes_launch_cfg_t *cfg,
                    const DeviceInfo &di)
{
    Shape sh = default_shape(variant, key_bits, len, aligned, di);
    if (cfg && sh.variant == AES_VARIANT_TTABLE && other_shape(*cfg, sh))
        sh = explicit_base(key_bits, len, di);
    if (cfg) {
        if (cfg->blocks_per_lane) sh.bpl = cfg->blocks_per_lane;
        if (cfg->wg_size) sh.wg = cfg->wg_size;
        if (cfg->grid) sh.grid = cfg->grid;
        if (cfg->lds_copies) sh.copies = cfg->lds_copies;
        if (cfg->lds_tables) sh.tables = cfg->lds_tables;
    }
    // 64 copies exist only of two tables; a T-table shape always names both.
    if (sh.variant == AES_VARIANT_TTABLE) {
        if (sh.copies == 64)
            sh.tables = 2;
        else if (sh.tables == 0)
            sh.tables = 4;
    }
    if (sh.variant != AES_VARIANT_TTABLE) {
        sh.copies = 0;
        sh.tables = 0;
    }
    if (sh.variant == AES_VARIANT_VPERM)
        sh.bpl = 1;     // one block per lane, whatever cfg asks
    clamp_grid(&sh, len);
    // First-chunk mode of the T-table kernel: cfg's, else the tuned entry's
    // or the rule's (mode 2 up to 4 MiB) where the shape is built for it.
    // Per-wave first-chunk group constants pay off when two workgroups with
    // the 64 KiB image share each CU (8 MiB AES-128: 7.64-7.69 against
    // 7.74-7.78 us); other shapes fall back to wave 0 computing them.
    const int tuned = sh.wave_groups;
    sh.wave_groups = kFirstWave0;
    if (sh.variant == AES_VARIANT_TTABLE) {
        if (cfg && cfg->wave_groups)
            sh.wave_groups = cfg->wave_groups == 3 ? kFirstWave0 : cfg->wave_groups;
        else if (tuned >= 0 && first_chunk_mode_ok(tuned, sh.copies, sh.tables, sh.bpl, sh.wg))
            sh.wave_groups = tuned;
        else if (sh.copies == 32 && sh.tables == 2 && sh.bpl == 2 && sh.wg <= 512 && sh.grid >= 2 * di.num_cus)
            sh.wave_groups = kFirstPerWave;
    }
    return sh;
}

}  // namespace

extern "C" int aes_ctr_launch_shape(int key_bits, size_t len, const aes_launch_cfg_t *cfg, aes_launch_cfg_t *out)
{
    if (!out || (key_bits != 128 && key_bits != 256))
        return AES_EINVAL;
    int variant;
    int rc = check_cfg(cfg, &variant);
    if (rc != AES_OK)
        return rc;
    DeviceInfo di;
    if ((rc = device_info(&di)) != AES_OK)
        return rc;
    const Shape sh = resolve_shape(variant, key_bits, len ? len : 1, true, cfg, di);
    *out = aes_launch_cfg_t{};
    out->variant = sh.variant;
    out->blocks_per_lane = sh.bpl;
    out->wg_size = sh.wg;
    out->grid = sh.grid;
    out->lds_copies = sh.copies;
    out->lds_tables = sh.tables;
    if (sh.variant == AES_VARIANT_TTABLE &&
        !first_chunk_mode_ok(sh.wave_groups, sh.copies, sh.tables, sh.bpl, sh.wg))
        return AES_EINVAL;
    out->wave_groups = sh.wave_groups;
    return AES_OK;
}

extern "C" int aes_ctr_crypt_cfg(const aes_sched_t *sched, const uint8_t nonce[12], uint32_t ctr0,
                                 const void *in, void *out, size_t len, const aes_launch_cfg_t *cfg,
                                 void *stream)
{
    int rc = check_sched(sched);
    if (rc != AES_OK)
        return rc;
    if (!nonce)
        return AES_EINVAL;
    if ((rc = check_buffers(in, out, len)) != AES_OK)
        return rc;
    int variant;
    if ((rc = check_cfg(cfg, &variant)) != AES_OK)
        return rc;
    if (len == 0)
        return AES_OK;

    DeviceInfo di;
    if ((rc = device_info(&di)) != AES_OK)
        return rc;
    const bool aligned = ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    const Shape sh = resolve_shape(variant, sched->key_bits, len, aligned, cfg, di);

    hipStream_t st = static_cast<hipStream_t>(stream);
    if (sh.variant == AES_VARIANT_VPERM) {
        VpArgs va;
        make_vperm_args(*sched, nonce, ctr0, in, out, len, &va);
        return launch_ctr_vperm(va, sched->nr, sh, st);
    }
    KeyMaterial km;
    make_key_material(*sched, nonce, &km);
    CtrArgs a{};
    a.in = static_cast<const uint8_t *>(in);
    a.out = static_cast<uint8_t *>(out);
    a.len = len;
    a.ctr0 = ctr0;
    a.x0 = km.x0;
    memcpy(a.k1, km.k1, sizeof(a.k1));
    memcpy(a.rk, km.rk, sizeof(a.rk));
    if (sh.variant == AES_VARIANT_BITSLICE)
        return launch_ctr_bitslice(a, km.nr, sh, st);
    // Quads and pairs of lanes have grids and workgroups of their own, so they
    // are for callers who leave the shape to the library.
    if (!names_shape(cfg)) {
        if (quad_shape(sh, len, di.num_cus))
            return launch_ctr_quad(a, km.nr, st);
        if (pair_shape(sh, len, di.num_cus))
            return launch_ctr_pair(a, km.nr, st);
    }
    if (bulk_shape(sh, len))
        return launch_ctr_bulk(a, km.nr, sh, st);
    return launch_ctr_ttable(a, km.nr, sh, st);
}

extern "C" int aes_ctr_crypt(const aes_sched_t *sched, const uint8_t nonce[12], uint32_t ctr0,
                             const void *in, void *out, size_t len, void *stream)
{
    return aes_ctr_crypt_cfg(sched, nonce, ctr0, in, out, len, nullptr, stream);
}
