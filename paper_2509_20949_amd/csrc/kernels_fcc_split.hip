// kernels_fcc_split.hip -- the FCC sweep kernel for launches with few blocks:
// four lanes per trial and four wavefronts per block (the BCC counterpart,
// kernels_split.hip, says why).
//
// A launch of few blocks with one wave per block (kernels_fcc.hip) takes 108
// dependent rounds, each 50 byte reads among some 250 instructions one after
// the other, from code specialised on the partner's direction that does not
// fit the instruction cache.  Here a lane counts half
// of the site's or of the partner's neighbourhood, 21 cells.
//
// Image.  Sites are addressed by their doubled local coordinates (X, Y, Z):
//   (X + 4) / 2 + kFY (Y + 3) + kFZ (Z + 3),  X, Y, Z in -3 .. 26
// (X's parity follows from Y and Z).  A displacement then has one offset for
// all four sublattices, but for +1 more where dx is odd and X is odd: cells at
// odd dx are read from a second base, and one copy of the code serves every
// sublattice, partner and sign.
//
// Halves (sigma = +-1): the cells at dz = sigma and 2 sigma, and of the plane
// dz = 0 the cells (+-1, sigma, 0), (2 sigma, 0, 0) and (0, 2 sigma, 0):
// translates of each other shell by shell.
//
// No barrier separates the rounds of one z residue: in doubled coordinates a
// trial reads within 3 of its site and changes within 1 per axis, and the
// waves split the round's cells by z, 6 apart for one sublattice and at least
// 5 for two.
//
// Measured (K = 5, S = 3, 24^3 cells, 1 block per colour): 41 us per launch
// against 75 with one wave per block (113 before that kernel loaded the site
// and its partner first); a round takes about 750 cycles, some
// 420 of them issue.
#include <type_traits>

#include "split_trial.h"

namespace smcx {
namespace fsplit {

using split::LaneRole;
constexpr int kFY = 16, kFZ = 488;               // with the lane map below a read takes 3.1 LDS cycles (bank model)
constexpr int kImage = 30 * kFZ;
constexpr int kF = 6, kK = 5;                    // bits per species field, species
constexpr uint32_t kFieldBias = 32u * (1u | 1u << 6 | 1u << 12 | 1u << 18 | 1u << 24);

// sublattice offsets (doubled): (0,0,0), (1,1,0), (1,0,1), (0,1,1)
__device__ __forceinline__ constexpr int sx(int b) { return b == 1 || b == 2; }
__device__ __forceinline__ constexpr int sy(int b) { return b == 1 || b == 3; }
__device__ __forceinline__ constexpr int sz(int b) { return b >= 2; }
// LDS position of site b of local cell (lx, ly, lz)
__device__ __forceinline__ int site(int b, int lx, int ly, int lz)
{
    return lx + 2 + kFY * (2 * ly + sy(b) + 3) + kFZ * (2 * lz + sz(b) + 3);
}

// One trial: p the lane's centre (site or partner), odd its X parity.
template <int SMAX, int MODE>
__device__ __forceinline__ int32_t trial(uint8_t* p, int odd, const LaneRole& r, float lo, const uint32_t* u_at,
                                         const int32_t* wtab, const double* tab, uint32_t& nacc)
{
    const uint32_t own = *p;
    // bases (e: cells at even dx, o: at odd dx = -1, +1 -> -1, 0), less what
    // keeps their offsets non-negative
    const uint8_t* o = p + odd;
    const int z1 = r.half * kFZ, y1 = r.half * kFY;
    const uint8_t *ze = p + (z1 - kFY - 1), *zo = o + (z1 - 2 * kFY - 1);
    const uint8_t *zze = p + 2 * z1, *zzo = o + (2 * z1 - kFY - 1);
    const uint8_t *yo = o + (y1 - 1), *yy = p + 2 * y1, *xx = p + r.half;
    constexpr int E0 = kFY + 1, O0 = 2 * kFY + 1, Z0 = kFY + 1;   // the bases' zero
    uint32_t n1[6], n2[3], n3[12];
    n1[0] = zo[O0];
    n1[1] = zo[O0 - 1];
    n1[2] = ze[E0 + kFY];
    n1[3] = ze[E0 - kFY];
    n1[4] = yo[1];
    n1[5] = yo[0];
    if constexpr (SMAX >= 2) {
        n2[0] = zze[0];
        n2[1] = xx[0];
        n2[2] = yy[0];
    }
    if constexpr (SMAX >= 3) {
        n3[0] = ze[E0 + kFY + 1];
        n3[1] = ze[E0 + kFY - 1];
        n3[2] = ze[E0 - kFY + 1];
        n3[3] = ze[E0 - kFY - 1];
        n3[4] = zo[O0 + 2 * kFY];
        n3[5] = zo[O0 + 2 * kFY - 1];
        n3[6] = zo[O0 - 2 * kFY];
        n3[7] = zo[O0 - 2 * kFY - 1];
        n3[8] = zzo[Z0 + kFY];
        n3[9] = zzo[Z0 + kFY - 1];
        n3[10] = zzo[Z0 - kFY];
        n3[11] = zzo[Z0 - kFY - 1];
    }
    return split::finish_trial<kK, SMAX, kF, MODE>(p, own, n1, n2, n3, r, lo, u_at, wtab, tab, nacc);
}

}  // namespace fsplit

// One block per workgroup of 4 waves; n workgroups: the blocks of a single
// lattice, or kWavesPerGroupFcc per work item.
template <int SMAX>
__global__ __launch_bounds__(4 * kWave)
void sweep_fcc_split_kernel(const DevLattice* __restrict__ lats, const WorkItem* __restrict__ items, int n, int t,
                            int colour)
{
    using namespace fsplit;
    constexpr int kWBytes = wplanes(kK, SMAX) * kPlane * 4;
    // per wave, for one z residue: the draws of its 9 classes x 16 cells x 4
    // sublattices and their edges, at ((16 class + cell) * 4 + sublattice)
    constexpr int kDraws = 9 * 16 * 4;
    __shared__ __attribute__((aligned(16))) uint8_t s_mem[kWBytes + 4 * 8 * kDraws + kImage];
    int32_t* s_w = (int32_t*)s_mem;
    uint8_t* lat = s_mem + kWBytes + 4 * 8 * kDraws;

    const int wave = wave_id();
    const int lane = threadIdx.x % kWave;
    uint32_t* draws = (uint32_t*)(s_mem + kWBytes) + wave * 2 * kDraws;
    float* edges = (float*)(draws + kDraws);
    const int grp = xcd_group(n);
    if (grp < 0) return;
    int li = 0, f = grp;
    if (items) {
        const WorkItem it = items[grp / kWavesPerGroupFcc];
        li = it.lattice;
        f = it.first_block + grp % kWavesPerGroupFcc;
    }
    const DevLattice& D = lats[li];
    if (f >= D.blocks_per_colour) return;   // the whole workgroup
    const uint32_t s = D.sweep0 + (uint32_t)t;
    int ti = (int)(s - D.tab_s0);
    ti = ti < 0 ? 0 : (ti >= D.n_tabs ? D.n_tabs - 1 : ti);
    const double* g_tab = D.tabs + (size_t)ti * kTab;
    const float ln2kT = (float)g_tab[kTabLn2kT];
    const uint32_t k0 = D.key[0], k1 = D.key[1];

    // the weight planes' words, on their way while the block is set up
    constexpr int kWords = wplanes(kK, SMAX) * kPlane, kWPer = (kWords + 4 * kWave - 1) / (4 * kWave);
    int32_t wword[kWPer];
#pragma unroll
    for (int w = 0; w < kWPer; ++w) {
        const int k = w * 4 * kWave + (int)threadIdx.x, row = k % kPlane;
        wword[w] = k < kWords && row < kK * kK ? D.wtab[row * wrow(kK, SMAX) + k / kPlane] : 0;
    }

    // partner of every (colour, sub-colour q) set of this sweep, from
    // r = Philox(key, (q, 0, s, c + 64)): sublattice = the k-th other than the
    // set's own, k = (r0 * 3) >> 32, signs = bits 30 and 31 of r1.  Lane q
    // (q - 64) of part[0] (part[1]) holds 2 * offset + (dx odd).  The origin
    // shift (0, 0, s, 8) takes an idle lane of the second call.
    int part[2];
    uint32_t shift[3];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int q = 64 * h + lane;
        const bool own_shift = h == 1 && lane == 63;
        uint32_t r[4] = {own_shift ? 0u : (uint32_t)q, 0u, s, own_shift ? 8u : (uint32_t)colour + 64u};
        philox4x32_10(r, k0, k1);
        if (h == 1)
            for (int a = 0; a < 3; ++a) shift[a] = (uint32_t)__builtin_amdgcn_readlane((int)r[a], 63);
        const int b = q & 3, k = (int)(((uint64_t)r[0] * 3u) >> 32), bp = k + (k >= b ? 1 : 0);
        const int s0 = r[1] >> 30 & 1 ? 1 : -1, s1 = r[1] >> 31 ? 1 : -1;   // first and second differing axis
        const bool xd = sx(b) != sx(bp), yd = sy(b) != sy(bp), zd = sz(b) != sz(bp);
        const int off = (xd ? (s0 - 1) / 2 + sx(b) : 0) + (yd ? kFY * (xd ? s1 : s0) : 0) + (zd ? kFZ * s1 : 0);
        part[h] = 2 * off + (xd ? 1 : 0);
    }

    const int hx = D.nb[0] >> 1, hy = D.nb[1] >> 1;
    const int kx = 2 * (f % hx) + (colour & 1);
    const int ky = 2 * ((f / hx) % hy) + ((colour >> 1) & 1);
    const int kz = 2 * (f / (hx * hy)) + ((colour >> 2) & 1);
    const int Lx = D.L[0], Ly = D.L[1], Lz = D.L[2];
    const int ox = (int)(((uint64_t)shift[0] * (uint32_t)Lx) >> 32);
    const int oy = (int)(((uint64_t)shift[1] * (uint32_t)Ly) >> 32);
    const int oz = (int)(((uint64_t)shift[2] * (uint32_t)Lz) >> 32);
    const int x0 = block_lo(kx, Lx, D.nb[0]), wx = block_lo(kx + 1, Lx, D.nb[0]) - x0;
    const int y0 = block_lo(ky, Ly, D.nb[1]), wy = block_lo(ky + 1, Ly, D.nb[1]) - y0;
    const int z0 = block_lo(kz, Lz, D.nb[2]), wz = block_lo(kz + 1, Lz, D.nb[2]) - z0;
    const int gx0 = wrap_add(x0 + ox, Lx), gy0 = wrap_add(y0 + oy, Ly), gz0 = wrap_add(z0 + oz, Lz);
    uint8_t* __restrict__ g = D.species;
    const bool dot_codes = D.drop_last == kWtabDot;

    // Draws of z residue rz for this wave's cells (iz = wave): lane -> cell
    // lane & 15, class (lane >> 4) + 4 n; one call per cell, word b for site b.
    auto draw = [&](int rz) {
        const int ix = lane & 3, iy = (lane >> 2) & 3;
        uint32_t gz = (uint32_t)(gz0 + 3 * wave + rz);
        gz = min(gz, gz - (uint32_t)Lz);
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            const int c = (lane >> 4) + 4 * n, rx = c % 3, ry = c / 3;
            uint32_t gx = (uint32_t)(gx0 + 3 * ix + rx), gy = (uint32_t)(gy0 + 3 * iy + ry);
            gx = min(gx, gx - (uint32_t)Lx);
            gy = min(gy, gy - (uint32_t)Ly);
            const uint64_t cell = ((uint64_t)gz * (uint32_t)Ly + gy) * (uint32_t)Lx + gx;
            uint32_t u[4] = {(uint32_t)cell, (uint32_t)(cell >> 32), s, (uint32_t)colour};
            philox4x32_10(u, k0, k1);
            const bool valid = (3 * ix < wx - rx) & (3 * iy < wy - ry) & (3 * wave < wz - rz);
            if (c < 9) {
                const int at = (16 * c + (lane & 15)) * 4;
                *(uint4*)(draws + at) = make_uint4(u[0], u[1], u[2], u[3]);
                *(float4*)(edges + at) =
                    make_float4(split::accept_edge(u[0], ln2kT, valid), split::accept_edge(u[1], ln2kT, valid),
                                split::accept_edge(u[2], ln2kT, valid), split::accept_edge(u[3], ln2kT, valid));
            }
        }
    };

    // ---- stage block + halo: one cell (4 sublattice bytes, one dword) per
    // lane, 4 rows of a plane per instruction, 4 planes per wave; all 16 loads
    // are in flight while the first draws are made ----
    {
        const int lx = (lane & 15) - 2;
        const bool okx = lx <= wx + 1;
        const int gx = wrap_add(gx0 + (okx ? lx : -2), Lx);
        const int lz0 = 4 * wave - 2;
        uint32_t v16[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int ly = min((lane >> 4) + 4 * (u & 3) - 2, wy + 1), lz = min(lz0 + (u >> 2), wz + 1);
            const int gy = wrap_add(gy0 + ly, Ly), gz = wrap_add(gz0 + lz, Lz);
            v16[u] = gload<uint32_t>(g + 4 * (((size_t)gz * Ly + gy) * Lx + gx));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int w = 0; w < kWPer; ++w) {
            const int k = w * 4 * kWave + (int)threadIdx.x;
            if (k < kWords) s_w[k] = wword[w];
        }
        draw(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int ly = (lane >> 4) + 4 * (u & 3) - 2, lz = lz0 + (u >> 2);
            if (!okx || ly > wy + 1 || lz > wz + 1) continue;
            const uint32_t v = v16[u];
            const uint32_t c = dot_codes ? encode4_dot<kK>(v) : (v << 5) + (v << 2) + (v << 1);   // else (6 + 32) * species
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (lx >= -1 - sx(b) && lx <= wx + 1 - sx(b) && ly >= -1 - sy(b) && ly <= wy + 1 - sy(b) &&
                    lz >= -1 - sz(b) && lz <= wz + 1 - sz(b))
                    lat[site(b, lx, ly, lz)] = (uint8_t)(c >> (8 * b));
        }
    }

    // ---- 27 residue classes x 4 sublattices = 108 rounds ----
    // Lane -> (trial, part): bits 0, 1 the part, 2 and 5 ix, 3 and 4 iy; iz =
    // wave.
    const int ix = (lane >> 2 & 1) | (lane >> 4 & 2), iy = lane >> 3 & 3;
    const bool work = 3 * wave < wz;   // some lane of the wave has sites
    int64_t dEsum = 0;
    uint32_t nacc = 0;
    __syncthreads();
    auto all_rounds = [&](auto mode_tag) {
        constexpr int MODE = decltype(mode_tag)::value;
        const LaneRole role = split::lane_role(lane, MODE == kWtabDot ? 0x20202020u : kFieldBias);
#pragma nounroll
        for (int rz = 0; rz < 3; ++rz) {
            if (rz) __syncthreads();
            if (!work) continue;   // (such a wave only meets the barriers)
            if (rz) draw(rz);
            __builtin_amdgcn_wave_barrier();
#pragma nounroll
            for (int c = 0; c < 9; ++c) {
                const int rx = c % 3, ry = c / 3, q0 = 4 * (9 * rz + c);
                const int word = (16 * c + 4 * iy + ix) * 4;
                const float4 lo = *(const float4*)(edges + word);
                uint8_t* at = lat + site(0, 3 * ix + rx, 3 * iy + ry, 3 * wave + rz);
                const int pv = q0 < 64 ? part[0] : part[1];
                auto step = [&](auto bc, float edge) {
                    constexpr int b = decltype(bc)::value;
                    const int pb = __builtin_amdgcn_readlane(pv, q0 + b);   // (lane q0 + b modulo 64)
                    uint8_t* p = at + (sy(b) * kFY + sz(b) * kFZ) + __mul24(pb >> 1, role.at_partner);
                    const int odd = sx(b) ^ (pb & role.at_partner);
                    const int32_t d = trial<SMAX, MODE>(p, odd, role, edge, draws + word + b, s_w, g_tab, nacc);
                    __builtin_amdgcn_wave_barrier();
                    return d;
                };
                int32_t d = step(std::integral_constant<int, 0>{}, lo.x);
                d += step(std::integral_constant<int, 1>{}, lo.y);
                dEsum += (int64_t)d;   // (two changes at a time stay inside 32 bits)
                d = step(std::integral_constant<int, 2>{}, lo.z);
                d += step(std::integral_constant<int, 3>{}, lo.w);
                dEsum += (int64_t)d;
            }
        }
    };
    if (dot_codes)
        all_rounds(std::integral_constant<int, kWtabDot>{});
    else
        all_rounds(std::integral_constant<int, kWtabFull>{});
    __syncthreads();

    // ---- write back: sublattice b over cells -SUB[b][a] .. w_a - SUB[b][a] ----
    {
        const int lx = (lane & 15) - 1;
        const bool okx = lx <= wx;
        const int lxc = okx ? lx : 0;
        const int gx = wrap_add(gx0 + lx, Lx);
        for (int lz = wave - 1; lz <= wz; lz += 4) {
            uint32_t c[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int lyc = min((lane >> 4) + 4 * u - 1, wy);
#pragma unroll
                for (int b = 0; b < 4; ++b) c[u][b] = lat[site(b, lxc, lyc, lz)];
            }
            const int gz = wrap_add(gz0 + lz, Lz);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ly = (lane >> 4) + 4 * u - 1;
                if (!okx || ly > wy) continue;
                bool v[4];
                uint32_t e = 0u;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    v[b] = lx >= -sx(b) && lx <= wx - sx(b) && ly >= -sy(b) && ly <= wy - sy(b) && lz >= -sz(b) &&
                           lz <= wz - sz(b);
                    e |= decode(c[u][b]) << (8 * b);
                }
                if (!(v[0] || v[1] || v[2] || v[3])) continue;
                uint8_t* q = g + 4 * (((size_t)gz * Ly + wrap_add(gy0 + ly, Ly)) * Lx + gx);
                if (v[0] && v[1] && v[2] && v[3]) {
                    gstore<uint32_t>(q, e);
                } else {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if (v[b]) gstore<uint8_t>(q + b, (uint8_t)(e >> (8 * b)));
                }
            }
        }
    }

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

hipError_t launch_sweep_split_fcc(const DevLattice* d_lat, const WorkItem* d_items, int n, int t, int colour, int smax,
                                  hipStream_t stream)
{
    const dim3 grid(xcd_grid(n)), block(4 * kWave);
    switch (smax) {
    case 1: hipLaunchKernelGGL((sweep_fcc_split_kernel<1>), grid, block, 0, stream, d_lat, d_items, n, t, colour); break;
    case 2: hipLaunchKernelGGL((sweep_fcc_split_kernel<2>), grid, block, 0, stream, d_lat, d_items, n, t, colour); break;
    case 3: hipLaunchKernelGGL((sweep_fcc_split_kernel<3>), grid, block, 0, stream, d_lat, d_items, n, t, colour); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace smcx
