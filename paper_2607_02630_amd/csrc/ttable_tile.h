// ttable_tile.h -- a wave's run over consecutive blocks of one message, shared
// by the batch kernel (ctr_batch.hip) and the kernel for large messages
// (ctr_bulk.hip).
#pragma once

#include "ttable_device.h"

namespace aesctr {
namespace {

// ---- A run of one message's blocks on one wave -----------------------------
//
// A message is laid out by position, block j at position j + message_shift(ctr0),
// so that 64 positions from a multiple of 64 have counters from a multiple of
// 64 and share their top three bytes.  For a lane that takes position p0 + 64 k
// + lane in step k, the counter's low byte then repeats every four steps, and
// rounds 1-2 split into a part that depends on it alone (lane_consts, four
// steps' worth in 16 registers) and one that is the same for the step's 64
// counters (group_consts_lds for 64 consecutive groups at a time, a lane each,
// handed over with v_readlane): four XORs per block where the wave's scalar
// constants took 5 lookups, 15 VALU instructions and a chain of scalar loads
// per step (main loop of the four-table kernel by its listing, AES-128: 128 lookups
// and 202 VALU instructions per block, 133 and 238 before).
__host__ __device__ __forceinline__ uint32_t message_shift(uint32_t ctr0) { return ctr0 & 63u; }

// Round 2 of every column without its group constant, for counters whose low
// byte is `low`.
template <int LAYOUT>
__device__ __forceinline__ void lane_consts(const TTable<LAYOUT> &tt, const CtrArgs &a, uint32_t low, uint32_t L[4])
{
    const uint32_t s10 = a.k1[0] ^ tt.template get<3, 3>((low << 24) ^ a.x0);
    L[0] = tt.template get<0, 0>(s10);
    L[1] = tt.template get<3, 3>(s10);
    L[2] = tt.template get<2, 2>(s10);
    L[3] = tt.template get<1, 1>(s10);
}

// Part of a message, in positions counted from its start (in 32 bits: the round
// keys leave few scalar registers): [lo, hi) are whole blocks of the message,
// `odd` is its partial block, or ~0.  in, out: the memory of position 0.
struct Span {
    const uint8_t *in;
    uint8_t *out;
    uint32_t lo, hi, odd;
};

// The part [p0, p1) of message a; p1 - p0 is below 2^31.
__device__ __forceinline__ Span message_span(const CtrArgs &a, uint32_t shift, uint64_t p0, uint64_t p1)
{
    const uint64_t end = (a.len >> 4) + shift;    // position of the partial block
    const int64_t base = 16 * (static_cast<int64_t>(p0) - shift);
    Span s;
    s.in = a.in + base;
    s.out = a.out + base;
    s.lo = p0 < shift ? static_cast<uint32_t>(shift - p0) : 0;
    s.hi = static_cast<uint32_t>((end < p1 ? end : p1) - p0);
    s.odd = (a.len & 15) != 0 && end < p1 ? s.hi : ~0u;
    return s;
}

// 64 N positions from q of span sp: rounds 1-2 from the lane's constants L and
// the group constants G of each 64, rounds 3 to Nr, and the data.  The keystream
// of the partial block goes into part.
template <int NR, int LAYOUT, int N>
__device__ __forceinline__ void span_step(const TTable<LAYOUT> &tt, const CtrArgs &a, const uint32_t *krot,
                                          const Span &sp, uint32_t q, uint32_t lane, const uint32_t (*L)[4],
                                          const uint32_t (&G)[N][4], u32x4 &part)
{
    const bool whole = q >= sp.lo && q + 64 * N <= sp.hi;
    u32x4 d[N];
    if (whole) {
#pragma unroll
        for (int b = 0; b < N; ++b) d[b] = load_block(sp.in, q + 64 * b + lane);
    } else {
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const uint32_t i = q + 64 * b + lane;
            if (i >= sp.lo && i < sp.hi)
                d[b] = load_block(sp.in, i);
        }
    }
    uint32_t s[N][4], o[N][4];
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) s[b][c] = G[b][c] ^ L[b][c];
#pragma unroll
    for (int r = 3; r < NR; ++r) {
#pragma unroll
        for (int b = 0; b < N; ++b)
            tt.round(s[b], o[b], &a.rk[4 * r], &krot[4 * r]);
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) s[b][c] = o[b][c];
    }
#pragma unroll
    for (int b = 0; b < N; ++b)
        tt.last_round(s[b], o[b], &a.rk[4 * NR]);
    if (whole) {
#pragma unroll
        for (int b = 0; b < N; ++b)
            store_block(sp.out, q + 64 * b + lane, d[b] ^ u32x4{o[b][0], o[b][1], o[b][2], o[b][3]});
    } else {
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const uint32_t i = q + 64 * b + lane;
            const u32x4 ks = {o[b][0], o[b][1], o[b][2], o[b][3]};
            if (i >= sp.lo && i < sp.hi)
                store_block(sp.out, i, d[b] ^ ks);
            if (i == sp.odd)
                part ^= ks;
        }
    }
}

// Positions [p0, p1) of message a, p0 a multiple of 64 and p1 - p0 below 2^31,
// N x 64 of them per step; positions outside the message are left out.  krot:
// rotr(rk, 8) for the two-table layouts.
//
// SHIFTED: positions are as above.  Otherwise position j is block j: a tile then
// holds as many blocks as positions, which counts where a launch has just enough
// waves for its tiles, but the 64 counters of a step may span two groups, so their
// constants are chosen per lane (8 more v_readlane and 4 selects per 64 blocks).
template <int NR, int LAYOUT, int N, bool SHIFTED = true>
__device__ __forceinline__ void run_tile(const TTable<LAYOUT> &tt, const CtrArgs &a, const uint32_t *krot, uint64_t p0,
                                         uint64_t p1, uint32_t lane)
{
    static_assert(N == 1 || N == 2, "steps of 64 or 128 blocks");
    const uint32_t shift = SHIFTED ? message_shift(a.ctr0) : 0;
    const uint32_t n = static_cast<uint32_t>(p1 - p0);
    const uint32_t tail = static_cast<uint32_t>(a.len & 15);
    const Span sp = message_span(a, shift, p0, p1);
    const uint32_t first = a.ctr0 - shift + static_cast<uint32_t>(p0);    // counter of position p0
    u32x4 part = {0, 0, 0, 0};
    if (sp.odd != ~0u)
        part = load_partial(sp.in, sp.odd, tail);
    uint32_t L[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (64u * k < n)
            lane_consts(tt, a, first + 64 * k + lane, L[k]);
    uint32_t Gv[4];
    uint32_t window = SHIFTED ? ~0u : 0u - 64u;    // the 64 groups whose constants Gv holds, counted from p0's:
                                                   // their number / 64, or the first of them
    for (uint32_t q = 0; q < n;) {
#pragma unroll
        for (int k = 0; k < 4; k += N) {
            uint32_t G[N][4];
#pragma unroll
            for (int b = 0; b < N; ++b) {
                const uint32_t c0 = (first & 255u) + q + 64 * b, g = c0 >> 8;
                if constexpr (SHIFTED) {
                    if ((g >> 6) != window) {
                        window = g >> 6;
                        group_consts_lds(tt, a, ((first >> 8) + (window << 6) + lane) & 0xffffffu, Gv);
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        G[b][c] = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(Gv[c]), g & 63));
                } else {
                    const uint32_t g1 = (c0 + 63) >> 8;
                    if (g1 - window > 63) {
                        window = g;
                        group_consts_lds(tt, a, ((first >> 8) + window + lane) & 0xffffffu, Gv);
                    }
                    const bool next = (c0 & 255u) + lane > 255u;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int v = static_cast<int>(Gv[c]);
                        const int lo = __builtin_amdgcn_readlane(v, g - window);
                        const int hi = __builtin_amdgcn_readlane(v, g1 - window);
                        G[b][c] = static_cast<uint32_t>(next ? hi : lo);
                    }
                }
            }
            span_step<NR, LAYOUT, N>(tt, a, krot, sp, q, lane, &L[k], G, part);
            q += 64 * N;
            if (q >= n)
                break;
        }
    }
    if (sp.odd != ~0u && lane == (sp.odd & 63))
        store_partial(sp.out, sp.odd, tail, part);
}

}  // namespace
}  // namespace aesctr
