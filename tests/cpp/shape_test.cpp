// Reads launch requests "key_bits len variant blocks_per_lane wg_size grid
// lds_copies lds_tables wave_groups address" from stdin and prints for each what
// aes_ctr_crypt_cfg does with it: "status kernel blocks_per_lane wg grid copies
// tables mode", the shape as the kernel's launcher gets it.  The launchers are
// stand-ins that take what the kernels are built for.
#include <stdio.h>

#include "aesctr_internal.h"

namespace aesctr {
namespace {

const char *g_kernel = "-";
Shape g_shape;

int take(const char *kernel, const Shape &sh, bool ok = true)
{
    g_kernel = kernel;
    g_shape = sh;
    return ok ? AES_OK : AES_EINVAL;
}

bool small_shape(const Shape &sh, uint64_t len, uint64_t blocks_per_cu, int num_cus)
{
    const uint64_t blocks = (len + 15) / 16;
    g_shape = sh;
    return sh.copies == 32 && sh.tables == 2 && sh.wg == 256 && sh.bpl == 1 && sh.wave_groups == kFirstFull &&
           blocks <= blocks_per_cu * num_cus && blocks <= static_cast<uint64_t>(sh.grid) * sh.wg;
}

}  // namespace

int launch_ctr_ttable(const CtrArgs &, int, const Shape &sh, hipStream_t)
{
    const bool layout = (sh.copies == 32 && (sh.tables == 2 || sh.tables == 4)) || (sh.copies == 64 && sh.tables == 2);
    const bool chunk = (sh.wg == 256 || sh.wg == 512 || sh.wg == 1024) && (sh.bpl == 1 || sh.bpl == 2 || sh.bpl == 4);
    return take("ttable", sh, layout && chunk && sh.grid > 0 &&
                                  first_chunk_mode_ok(sh.wave_groups, sh.copies, sh.tables, sh.bpl, sh.wg));
}

bool quad_shape(const Shape &sh, uint64_t len, int num_cus) { return small_shape(sh, len, 128, num_cus); }
bool pair_shape(const Shape &sh, uint64_t len, int num_cus) { return small_shape(sh, len, 256, num_cus); }

bool bulk_shape(const Shape &sh, uint64_t len)
{
    return sh.copies == 32 && sh.tables == 4 && sh.wg == 1024 && sh.bpl == 2 && sh.wave_groups == kFirstWave0 &&
           len / 16 >= static_cast<uint64_t>(sh.grid) * 4096;
}

int launch_ctr_quad(const CtrArgs &, int, hipStream_t) { return take("quad", g_shape); }
int launch_ctr_pair(const CtrArgs &, int, hipStream_t) { return take("pair", g_shape); }
int launch_ctr_bulk(const CtrArgs &, int, const Shape &sh, hipStream_t) { return take("bulk", sh); }
int launch_ctr_bitslice(const CtrArgs &, int, const Shape &sh, hipStream_t) { return take("bitslice", sh); }
int launch_ctr_vperm(const VpArgs &, int, const Shape &sh, hipStream_t) { return take("vperm", sh); }
void make_vperm_args(const aes_sched_t &, const uint8_t *, uint32_t, const void *, void *, uint64_t, VpArgs *) {}

}  // namespace aesctr

int main()
{
    using namespace aesctr;
    int bits;
    unsigned long long len;
    aes_launch_cfg_t c{};
    const uint8_t key[32] = {}, nonce[12] = {};
    int address;
    while (scanf("%d %llu %d %d %d %d %d %d %d %d", &bits, &len, &c.variant, &c.blocks_per_lane, &c.wg_size, &c.grid,
                 &c.lds_copies, &c.lds_tables, &c.wave_groups, &address) == 10) {
        void *buf = reinterpret_cast<void *>((uintptr_t(1) << 40) + address);
        aes_sched_t s;
        if (aes_expand_key(key, bits, &s) != AES_OK)
            return 1;
        g_kernel = "-";
        const int rc = aes_ctr_crypt_cfg(&s, nonce, 1, buf, buf, len, &c, nullptr);
        printf("%d %s %d %d %d %d %d %d\n", rc, g_kernel, g_shape.bpl, g_shape.wg, g_shape.grid, g_shape.copies,
               g_shape.tables, g_shape.wave_groups);
    }
    return 0;
}
