// split_trial.h -- the lattice-independent part of a trial that four lanes
// share (kernels_split.hip, kernels_fcc_split.hip): counting a lane's cells,
// weighing them, summing the energy change over the lanes, the Metropolis
// decision and the swap.
#pragma once

#include "device_common.h"

namespace smcx {
namespace split {

// quad_perm controls: lanes 0..3 of every quad take the named lanes' values
constexpr int kSwap = 1 | 0 << 2 | 3 << 4 | 2 << 6;     // the other lane of the pair
constexpr int kSwap2 = 2 | 3 << 2 | 0 << 4 | 1 << 6;    // the other pair of the quad
template <int CTRL> __device__ __forceinline__ uint32_t quad(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}

// A lane's share of a trial: bit 0 of the lane says whose neighbourhood it
// counts (the site's or the partner's), bit 1 which half of it.  Lane 0 of the
// four adds the terms that enter once.
struct LaneRole {
    int at_partner;      // 1 on lanes that count the partner's neighbourhood
    int half;            // +1 or -1: the half of the neighbourhood
    uint32_t lead;       // all ones on the lead lane
    uint32_t bias;       // the histogram fields' offset, on the lead lane
};
__device__ __forceinline__ LaneRole lane_role(int lane, uint32_t bias)
{
    LaneRole r;
    r.at_partner = lane & 1;
    r.half = lane & 2 ? 1 : -1;
    r.lead = (lane & 3) == 0 ? ~0u : 0u;
    r.bias = r.lead & bias;
    return r;
}

// acc + sum over shells and fields (F bits each) of field(s, p) *
// w[s*KMAX + p], modulo 2^32 (the fields of one lane's partial counts).
template <int KMAX, int SMAX, int F, int NF>
__device__ __forceinline__ uint32_t weigh_fields(const uint32_t (&h)[kMaxS], const int32_t* w, uint32_t acc)
{
#pragma unroll
    for (int s = 0; s < SMAX; ++s)
#pragma unroll
        for (int p = 0; p < NF; ++p)
            acc = mad24((h[s] >> (F * p)) & ((1u << F) - 1u), w[(s * KMAX + p) * kPlane], acc);
    return acc;
}

// bias + sum of 1 << code over N codes, one shift-add each.  One asm block:
// between blocks of one chain the compiler puts a wait state, which here,
// one wave to a SIMD, costs an issue slot.
template <int N> __device__ __forceinline__ uint32_t count_all(uint32_t bias, const uint32_t (&c)[N])
{
    static_assert(N == 3 || N == 4 || N == 6 || N == 12, "neighbours of a lane per shell");
    uint32_t h;
    if constexpr (N == 12) {
        const uint32_t a[6] = {c[0], c[1], c[2], c[3], c[4], c[5]}, b[6] = {c[6], c[7], c[8], c[9], c[10], c[11]};
        h = count_all(count_all(bias, a), b);
    } else if constexpr (N == 3)
        asm("v_lshl_add_u32 %0, 1, %1, %4\n\tv_lshl_add_u32 %0, 1, %2, %0\n\tv_lshl_add_u32 %0, 1, %3, %0"
            : "=&v"(h) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(bias));
    else if constexpr (N == 4)
        asm("v_lshl_add_u32 %0, 1, %1, %5\n\tv_lshl_add_u32 %0, 1, %2, %0\n\tv_lshl_add_u32 %0, 1, %3, %0\n\t"
            "v_lshl_add_u32 %0, 1, %4, %0"
            : "=&v"(h) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(bias));
    else
        asm("v_lshl_add_u32 %0, 1, %1, %7\n\tv_lshl_add_u32 %0, 1, %2, %0\n\tv_lshl_add_u32 %0, 1, %3, %0\n\t"
            "v_lshl_add_u32 %0, 1, %4, %0\n\tv_lshl_add_u32 %0, 1, %5, %0\n\tv_lshl_add_u32 %0, 1, %6, %0"
            : "=&v"(h) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(c[4]), "v"(c[5]), "v"(bias));
    return h;
}

// The acceptance edge of a draw (Eq. (3)): a change dE with float(dE) <= lo
// is accepted without the threshold tables, one with float(dE) > lo + 16 is
// rejected, in between the table decides (accept_edges, device_common.h: lo
// is its lower edge, but never below 0, so that dE <= 0 passes; lo + 16 is
// its upper edge, or above it where lo was raised to 0).  Every edge of a draw u > 0 lies
// below 2^24 - 16.  A trial without a site gets -inf (always rejected), u = 0
// NaN (neither test passes: the table decides).
__device__ __forceinline__ float accept_edge(uint32_t u, float ln2kT, bool valid)
{
    float elo, ehi;
    accept_edges(u, ln2kT, elo, ehi);
    const float lo = u == 0u ? __builtin_nanf("") : fmaxf(elo, 0.0f);
    return valid ? lo : -__builtin_inff();
}

// The rest of a trial, from the code `own` at the lane's centre p (the site or
// its partner) and the codes of the lane's cells in shells 1 .. SMAX (loads
// in flight).  lo: the draw's edge, u_at: the draw itself in LDS.  Every lane
// of the trial takes the same decision; each stores the new code of its own
// centre.  Returns the accepted change.
template <int KMAX, int SMAX, int F, int MODE, int N1, int N2, int N3>
__device__ __forceinline__ int32_t finish_trial(uint8_t* p, uint32_t own, const uint32_t (&n1)[N1],
                                                const uint32_t (&n2)[N2], const uint32_t (&n3)[N3],
                                                const LaneRole& role, float lo, const uint32_t* u_at,
                                                const int32_t* wtab, const double* tab, uint32_t& nacc)
{
    constexpr bool DOT = MODE == kWtabDot;
    const uint32_t a = own >> 5;
    const uint32_t row4 = __umul24(a, 4u * KMAX) + quad<kSwap>(a << 2);   // row (own code, other code)
    const int32_t* w = (const int32_t*)((const uint8_t*)wtab + row4);
    // the byte-dot row is requested before the counting (the other forms load
    // theirs as they go)
    constexpr int NW = DOT ? 3 * SMAX + 1 : 1;
    int32_t wr[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) wr[k] = w[(DOT ? k : SMAX * KMAX) * kPlane];
    __builtin_amdgcn_sched_barrier(0);
    uint32_t h[kMaxS];
    h[0] = count_all(role.bias, n1);
    if constexpr (SMAX >= 2) h[1] = count_all(role.bias, n2);
    if constexpr (SMAX >= 3) h[2] = count_all(role.bias, n3);
    const uint32_t other = quad<kSwap>(own);
    uint32_t acc;
    if constexpr (DOT) {
        // the three base-256 digits of the folded weights, in chains of their own
        int32_t A0 = (int32_t)((uint32_t)wr[3 * SMAX] & role.lead), A1 = 0, A2 = 0;
#pragma unroll
        for (int s = 0; s < SMAX; ++s) {
            // (K <= 4: byte 3, where the last species' bit 31 lies, weighs nothing)
            const int32_t d = (int32_t)(KMAX == 5 ? h[s] & 0x7fffffffu : h[s]);
            A0 = __builtin_amdgcn_sdot4(d, wr[3 * s + 0], A0, false);
            A1 = __builtin_amdgcn_sdot4(d, wr[3 * s + 1], A1, false);
            A2 = __builtin_amdgcn_sdot4(d, wr[3 * s + 2], A2, false);
        }
        acc = ((((uint32_t)A2 << 8) + (uint32_t)A1) << 8) + (uint32_t)A0;
    } else {
        acc = weigh_fields<KMAX, SMAX, F, MODE == kWtabDrop ? KMAX - 1 : KMAX>(
            h, w, (uint32_t)wr[0] & role.lead);
    }
    acc += quad<kSwap>(acc);
    acc += quad<kSwap2>(acc);
    const int32_t dE = (int32_t)acc;

    // Metropolis decision, Eq. (3); the exact test on the FP64 byte tables
    // only where a lane's change lies between its edges
    const float fdE = (float)dE;
    bool accept = fdE <= lo;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!accept & !(fdE > lo + 16.0f)) != 0, 0)) {
        // (the table decides as the edges do where those suffice; a lane
        // without a site keeps its edge's answer)
        const uint32_t u = *u_at;
        const int x = dE < 1 ? 1 : (dE > (1 << 24) - 1 ? (1 << 24) - 1 : dE);
        const uint8_t* tb = (const uint8_t*)tab;
        const double thr = (gload<double>(tb + 8 * (512 + (x >> 16))) * gload<double>(tb + 8 * (256 + ((x >> 8) & 255)))) *
                           gload<double>(tb + 8 * (x & 255));
        accept = !(lo < 0.0f) & ((dE <= 0) | ((dE < (1 << 24)) & ((double)u < thr)));
    }
    nacc += (accept & (own != other)) ? 1u : 0u;
    *p = (uint8_t)(accept ? other : own);   // (the two lanes of a centre store the same value)
    return accept ? dE : 0;                 // (0 for equal species: their row is zero)
}

}  // namespace split
}  // namespace smcx
