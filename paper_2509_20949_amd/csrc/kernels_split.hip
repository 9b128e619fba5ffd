// kernels_split.hip -- the BCC sweep kernel for launches with few blocks: four
// lanes per trial and four wavefronts per block.
//
// A colour launch lasts at least as long as one block's 54 rounds, which
// depend on each other through the lattice.  With one wavefront per block
// (kernels.hip) a wave alone on its SIMD issues a round's some 190
// instructions one after the other and waits for its LDS round trips.  Where a
// launch has fewer blocks than the chip has wave slots, that chain is its whole
// time.  Here four lanes count the two neighbourhoods of a trial
// side by side, so that a round is a third as many instructions of each wave,
// and the block's four waves run on the CU's four SIMDs.  Lane bit 0: the
// site's neighbourhood or the partner's.  Lane bit 1: one half of it or the
// other -- the lower or upper plane of the first shell and of the cells at
// dz = -+1, and the column x - 1 or x + 1 and one y neighbour of the middle
// plane: halves that are translates of each other shell by shell, so that
// all lanes read at common offsets from bases of their own.
// Every lane weighs its partial counts; the energy change is the sum over the
// trial's lanes (quad-permute adds).  A lane weighs with the row (own code,
// other code): the change of the partner's neighbourhood under b -> a is what
// the row (a, b) subtracts, and the rows are antisymmetric, so all lanes add.
//
// No barrier separates the rounds of one z residue.  In units of a/2 a trial
// reads cells within 3 of its site and changes cells within 1, per axis.  The
// waves split the round's 4 x 4 x 4 cells by z: sites of two waves are 6
// apart along z for one sublattice of one z residue and at least 5 for the
// two, so what a wave reads (3) and another changes (1) never meet, whatever
// round either is at.  Within a wave LDS operations complete in program
// order.  A barrier separates the three z residues.
//
// Measured (K = 5, S = 3, 64^3 cells, 27 blocks per colour): 19.5 us per
// launch against 31.5 with one wave per block (42.0 before that kernel carried
// a row's cells in registers); a round takes about 560 cycles,
// 330 of them issue, the rest two LDS round trips.  About 12,000 of the
// launch's 43,000 cycles are set-up, staging and write-back.
#include <type_traits>

#include "bcc_block.h"
#include "split_trial.h"

namespace smcx {

namespace split {

// LDS layout of the block image: with the lane map below, a byte read of a
// wave takes 2.9 LDS cycles on average over the sublattices, directions and
// offsets of a trial (a bank model; 4.3 with the one-wave kernel's pitches).
using Pitch = BccPitch<20, 303, 4573>;
constexpr int kX = 1, kY = Pitch::P, kZ = Pitch::PP;
// First-shell base from a corner site and from a body site; the neighbour
// e = ex + 2 ey + 4 ez is at base + ex + ey kY + ez kZ.
constexpr int kS1[2] = {Pitch::ARR, -Pitch::kBodyFromCorner};

// What a lane's place in its trial fixes for the whole launch.
struct LanePart {
    LaneRole role;
    int s1[2];           // first-shell base from the lane's centre, by the trial's sublattice
    int z, x, y;         // bases of the lane's z plane, x column and y neighbour, from its centre
};

template <int KMAX, bool DOT> __device__ __forceinline__ LanePart lane_part(int lane)
{
    LanePart c;
    c.role = lane_role(lane, DOT ? 0x20202020u
                           : Field<KMAX>::F == 5 ? 0x10u * (1u | 1u << 5 | 1u << 10 | 1u << 15 | 1u << 20 | 1u << 25) : 0u);
    const int up = c.role.half > 0 ? kZ : 0;
    c.s1[0] = kS1[c.role.at_partner] + up;
    c.s1[1] = kS1[1 - c.role.at_partner] + up;
    c.z = c.role.half * kZ - kY;   // (each less kY: their offsets 0 .. 2 kY are then immediates)
    c.x = c.role.half * kX - kY;
    c.y = c.role.half * kY;
    return c;
}

// One trial of sublattice SUB.  p: the lane's centre (the site or its
// partner), lo: the draw's edge, u_at: the draw itself in LDS.  Returns the
// accepted change.
// (Reading the next trial's centres ahead of this decision, with the two
// cells it may change put right afterwards, took 3 % longer: the selects cost
// the issue slots that the hidden LDS round trip gave.)
template <int KMAX, int SMAX, int SUB, int MODE>
__device__ __forceinline__ int32_t trial(uint8_t* p, const LanePart& c, float lo, const uint32_t* u_at,
                                         const int32_t* wtab, const double* tab, uint32_t& nacc)
{
    const uint32_t own = *p;
    // all neighbours before the first use
    const uint8_t *p1 = p + c.s1[SUB], *pz = p + c.z, *px = p + c.x, *py = p + c.y;
    uint32_t n1[4], n2[3], n3[6];
#pragma unroll
    for (int k = 0; k < 4; ++k) n1[k] = p1[(k & 1) + (k >> 1) * kY];
    if constexpr (SMAX >= 2) {
        n2[0] = pz[kY];
        n2[1] = px[kY];
        n2[2] = py[0];
    }
    if constexpr (SMAX >= 3) {
        n3[0] = pz[0];
        n3[1] = pz[kY - 1];
        n3[2] = pz[kY + 1];
        n3[3] = pz[2 * kY];
        n3[4] = px[0];
        n3[5] = px[2 * kY];
    }
    return finish_trial<KMAX, SMAX, Field<KMAX>::F, MODE>(p, own, n1, n2, n3, c.role, lo, u_at, wtab, tab, nacc);
}

}  // namespace split

// One block per workgroup of 4 waves; n workgroups: the blocks of a single
// lattice, or kWavesPerGroup per work item.
template <int KMAX, int SMAX, bool SLAB>
__global__ __launch_bounds__(4 * kWave)
void sweep_split_kernel(const DevLattice* __restrict__ lats, const WorkItem* __restrict__ items, int n, int t,
                        int colour)
{
    using split::Pitch;
    using split::kS1;
    constexpr int kWBytes = wplanes(KMAX, SMAX) * kPlane * 4;
    // the draws of the block's 27 x 64 x 2 trials and their edges (corner and
    // body of class m and cell c at (64 m + c) * 2), and the block image
    constexpr int kDraws = 28 * 64 * 2;
    __shared__ __attribute__((aligned(16))) uint8_t s_mem[kWBytes + 8 * kDraws + 2 * Pitch::ARR];
    int32_t* s_w = (int32_t*)s_mem;
    uint32_t* draws = (uint32_t*)(s_mem + kWBytes);
    float* edges = (float*)(draws + kDraws);
    uint8_t* lat = s_mem + kWBytes + 8 * kDraws;

    const int wave = wave_id();
    const int lane = threadIdx.x % kWave;
    const int grp = xcd_group(n);
    if (grp < 0) return;
    int li = 0, f = grp;
    if (items) {
        const WorkItem it = items[grp / kWavesPerGroup];
        li = it.lattice;
        f = it.first_block + grp % kWavesPerGroup;
    }
    const DevLattice& D = lats[li];
    if (f >= D.blocks_per_colour) return;   // the whole workgroup
    const uint32_t s = D.sweep0 + (uint32_t)t;
    int ti = (int)(s - D.tab_s0);
    ti = ti < 0 ? 0 : (ti >= D.n_tabs ? D.n_tabs - 1 : ti);
    const double* g_tab = D.tabs + (size_t)ti * kTab;
    const float ln2kT = (float)g_tab[kTabLn2kT];

    const uint32_t k0 = D.key[0], k1 = D.key[1];
    const BccDraws pb = bcc_draws(s, colour, k0, k1, lane);
    const BccBlock B = bcc_block<SLAB>(D, f, colour, pb);
    const bool dot_codes = KMAX <= 5 && D.drop_last == kWtabDot;
    // the weight planes' words (row-major table -> planes), on their way
    // while the block is set up
    constexpr int kWords = wplanes(KMAX, SMAX) * kPlane, kWPer = (kWords + 4 * kWave - 1) / (4 * kWave);
    int32_t wword[kWPer];
#pragma unroll
    for (int n = 0; n < kWPer; ++n) {
        const int k = n * 4 * kWave + (int)threadIdx.x, row = k % kPlane;
        wword[n] = k < kWords && row < KMAX * KMAX ? D.wtab[row * wrow(KMAX, SMAX) + k / kPlane] : 0;
    }
    int partner_off;   // lane q: the partner's offset in sub-colour q = 2m + b
    bcc_stage<KMAX, Pitch, SLAB, 4>(B, lat, lane, wave, dot_codes, [&] {
#pragma unroll
        for (int n = 0; n < kWPer; ++n) {
            const int k = n * 4 * kWave + (int)threadIdx.x;
            if (k < kWords) s_w[k] = wword[n];
        }
        // Draws: lane `lane` of wave w makes the calls of the block's cell
        // `lane` for class pairs w, w + 4, ..
        const int ix = lane & 3, iy = (lane >> 2) & 3, iz = lane >> 4;
        uint32_t base_lo, base_hi;
        bcc_base_cell<SLAB>(B, D.z_off, ix, iy, iz, base_lo, base_hi);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int k = n * 4 + wave;
            if (k >= 14) break;
            uint32_t w[4] = {base_lo, base_hi, s, (uint32_t)colour + 256u * (uint32_t)k};
            philox4x32_10(w, k0, k1);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int m = 2 * k + j;   // (class 27 does not exist: its words are not read)
                const int rx = m % 3, ry = (m / 3) % 3, rz = m / 9;
                const bool valid = (3 * ix < B.wx - rx) & (3 * iy < B.wy - ry) & (3 * iz < B.wz - rz);
                const int at = (64 * m + lane) * 2;
                *(uint2*)(draws + at) = make_uint2(w[2 * j], w[2 * j + 1]);
                *(float2*)(edges + at) = make_float2(split::accept_edge(w[2 * j], ln2kT, valid),
                                                     split::accept_edge(w[2 * j + 1], ln2kT, valid));
            }
        }
        const uint64_t yz = lane < 32 ? pb.yz_lo >> (2 * lane) : pb.yz_hi >> (2 * (lane & 31));
        partner_off = kS1[lane & 1] + (int)((pb.x >> lane) & 1) + (int)(yz & 1) * split::kY +
                      (int)((yz >> 1) & 1) * split::kZ;
    });

    // Lane -> (trial, part): a trial's four lanes are a quad; a wave holds
    // whole x and y lines of the round's 4 x 4 x 4 cells, the waves split them
    // along z.
    const int ix = (lane >> 2) & 3, iy = lane >> 4, iz = wave;
    const bool work = 3 * wave < B.wz;   // some lane of the wave has sites
    int64_t dEsum = 0;
    uint32_t nacc = 0;
    __syncthreads();

    auto all_rounds = [&](auto mode_tag) {
        constexpr int MODE = decltype(mode_tag)::value;
        const split::LanePart part = split::lane_part<KMAX, MODE == kWtabDot>(lane);
        int word = (16 * iz + 4 * iy + ix) * 2;
#pragma nounroll
        for (int rz = 0; rz < 3; ++rz) {
            if (rz) __syncthreads();
            if (!work) continue;   // (such a wave only meets the barriers)
            uint8_t* at = lat + ((3 * iz + 1 + rz) * split::kZ + (3 * iy + 1) * split::kY + (3 * ix + 1));
#pragma nounroll
            for (int ry = 0; ry < 3; ++ry, at += split::kY, word += 3 * 128) {
#pragma unroll
                for (int rx = 0; rx < 3; ++rx) {
                    const int q = 2 * (9 * rz + 3 * ry + rx);
                    const float2 lo = *(const float2*)(edges + word + 128 * rx);
                    const uint32_t* u = draws + word + 128 * rx;
                    uint8_t* p0 = at + rx + __mul24(__builtin_amdgcn_readlane(partner_off, q), part.role.at_partner);
                    uint8_t* p1 = at + rx + Pitch::kBodyFromCorner +
                                  __mul24(__builtin_amdgcn_readlane(partner_off, q + 1), part.role.at_partner);
                    int32_t d = split::trial<KMAX, SMAX, 0, MODE>(p0, part, lo.x, u, s_w, g_tab, nacc);
                    __builtin_amdgcn_wave_barrier();
                    d += split::trial<KMAX, SMAX, 1, MODE>(p1, part, lo.y, u + 1, s_w, g_tab, nacc);
                    __builtin_amdgcn_wave_barrier();
                    dEsum += (int64_t)d;   // (changes are below 2^29: two to a 32-bit sum)
                }
            }
        }
    };
    if constexpr (KMAX <= 5) {
        if (dot_codes)
            all_rounds(std::integral_constant<int, kWtabDot>{});
        else
            all_rounds(std::integral_constant<int, kWtabFull>{});
    } else {
        if (D.drop_last == kWtabDrop)
            all_rounds(std::integral_constant<int, kWtabDrop>{});
        else
            all_rounds(std::integral_constant<int, kWtabFull>{});
    }
    __syncthreads();
    bcc_write_back<Pitch, SLAB, 4>(B, lat, lane, wave);

    const bool lead = (lane & 3) == 0;
    uint64_t sum = lead ? (uint64_t)dEsum : 0u;
    uint32_t cnt = lead ? nacc : 0u;
#pragma unroll
    for (int o = 32; o >= 4; o >>= 1) {   // (lanes 4 apart: the lead lanes)
        const uint32_t lo = __shfl_xor((uint32_t)sum, o, kWave);
        const uint32_t hi = __shfl_xor((uint32_t)(sum >> 32), o, kWave);
        sum += (uint64_t)lo | ((uint64_t)hi << 32);
        cnt += __shfl_xor(cnt, o, kWave);
    }
    if (lane == 0) {
        unsigned long long* slot = (unsigned long long*)(D.state + ((4 * f + wave) % kSpread) * kSlotWords);
        if (sum) atomicAdd(slot, (unsigned long long)sum);
        if (cnt) atomicAdd(slot + 1, (unsigned long long)cnt);
    }
}

template <int KMAX, bool SLAB>
static hipError_t launch_s(const DevLattice* d_lat, const WorkItem* d_items, int n, int t, int colour, int smax,
                           hipStream_t stream)
{
    const dim3 grid(xcd_grid(n)), block(4 * kWave);
    switch (smax) {
    case 1: hipLaunchKernelGGL((sweep_split_kernel<KMAX, 1, SLAB>), grid, block, 0, stream, d_lat, d_items, n, t, colour); break;
    case 2: hipLaunchKernelGGL((sweep_split_kernel<KMAX, 2, SLAB>), grid, block, 0, stream, d_lat, d_items, n, t, colour); break;
    case 3: hipLaunchKernelGGL((sweep_split_kernel<KMAX, 3, SLAB>), grid, block, 0, stream, d_lat, d_items, n, t, colour); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool SLAB>
static hipError_t launch_k(const DevLattice* d_lat, const WorkItem* d_items, int n, int t, int colour, int kmax,
                           int smax, hipStream_t stream)
{
    switch (kmax) {
    case 2: return launch_s<2, SLAB>(d_lat, d_items, n, t, colour, smax, stream);
    case 3: return launch_s<3, SLAB>(d_lat, d_items, n, t, colour, smax, stream);
    case 4: return launch_s<4, SLAB>(d_lat, d_items, n, t, colour, smax, stream);
    case 5: return launch_s<5, SLAB>(d_lat, d_items, n, t, colour, smax, stream);
    case 6: return launch_s<6, SLAB>(d_lat, d_items, n, t, colour, smax, stream);
    case 8: return launch_s<8, SLAB>(d_lat, d_items, n, t, colour, smax, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_sweep_split(const DevLattice* d_lat, const WorkItem* d_items, int n, int t, int colour, int kmax,
                              int smax, hipStream_t stream, bool slab)
{
    return slab ? launch_k<true>(d_lat, d_items, n, t, colour, kmax, smax, stream)
                : launch_k<false>(d_lat, d_items, n, t, colour, kmax, smax, stream);
}

}  // namespace smcx
