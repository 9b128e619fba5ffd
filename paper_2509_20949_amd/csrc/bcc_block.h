// bcc_block.h -- one block of the shifted BCC block grid, as the sweep kernels
// hold it: its geometry, the LDS codes and offsets, the staging of block and
// halo from HBM and the write-back.  Shared by the kernel that gives a block
// one wavefront (kernels.hip) and the one that gives it several
// (kernels_split.hip): NW is the number of waves that share the block, w the
// calling wave's index among them.
#pragma once

#include "device_common.h"

namespace smcx {

// ---------------------------------------------------------------------------
// Species codes in LDS.  A site of species v is stored as (F + 32) * v, with
// F = 5 bits per species field when KMAX <= 6 and F = 4 otherwise: the low 5
// bits (the only bits a 32-bit shift reads) equal F * v, the top 3 bits equal
// v.  One shift-add per neighbour then counts species into packed fields.
template <int KMAX> struct Field { static constexpr int F = KMAX <= 6 ? 5 : 4; };

__device__ __forceinline__ uint32_t encode4(uint32_t species, int F)
{
    // up to four species bytes v_k -> bytes (F+32) v_k: no carries, as
    // (F+32) v <= 255 for every species the field width admits (all four
    // bytes are used, so no 24-bit multiply)
    return (species << 5) + species * (uint32_t)F;
}

// LDS pitches of a block image: row, plane, and bytes per sublattice array.
template <int P_, int PP_, int ARR_> struct BccPitch {
    static constexpr int P = P_, PP = PP_, ARR = ARR_;
    static constexpr int kBodyFromCorner = ARR + PP + P + 1;
    static_assert(PP >= 15 * P && ARR > 14 * PP + 14 * P + 14, "LDS array too small");
};
// The layout of the one-wave kernel (smcx_internal.h).
using WavePitch = BccPitch<kP, kPP, kArr>;

// LDS layout of one block (see smcx_internal.h): corner array at offset 0,
// body array at kArr.  Local cell (x, y, z):
//   corner: (z+1)*kPP + (y+1)*kP + (x+1)       x in -1..13
//   body:   kArr + (z+2)*kPP + (y+2)*kP + (x+2) x in -2..12


constexpr int kStageRows = 16;

// Geometry of one block of colour `colour` in sweep s (wave-uniform).
struct BccBlock {
    int Lx, Ly, Lz;
    int wx, wy, wz;          // block width per axis
    int gx0, gy0, gz0;       // global coordinate of local cell 0
    uint32_t LxLy;
    uint64_t plane_bytes;    // a plane of the lattice (or the slab buffer)
    uint64_t buf_bytes;
    bool plane32;            // a row's byte offsets fit 31 bits
    bool narrow;             // cell ids fit 32 bits and the 24-bit multiplier
    uint8_t* g;

    // plane of the lattice array that holds local z plane lz of the block:
    // periodic wrap, or on a slab the plane two further on (the array starts
    // with the two halo planes below the slab)
    template <bool SLAB> __device__ __forceinline__ int zplane(int lz) const
    {
        return SLAB ? gz0 + lz + 2 : wrap_add(gz0 + lz, Lz);
    }
};

// Draws shared by all blocks of (sweep s, colour): the origin shift of the
// sweep and the partner steps of the colour's rounds, all wave-uniform.  The x
// steps are bits q of x, the y and z steps bits 2q and 2q + 1 of yz_hi:yz_lo
// (sub-colour q = 2m + b).
struct BccDraws {
    uint32_t shift[3];
    uint64_t yz_lo, yz_hi, x;
};
// The three calls -- (0, 0, s, 8), (0, 0, s, 32 + colour), (0, 0, s, 40 +
// colour) -- run as one, in lanes 0, 1 and 2.
__device__ __forceinline__ BccDraws bcc_draws(uint32_t s, int colour, uint32_t k0, uint32_t k1, int lane)
{
    uint32_t c[4] = {0u, 0u, s, lane == 0 ? 8u : lane == 1 ? 32u + (uint32_t)colour : 40u + (uint32_t)colour};
    philox4x32_10(c, k0, k1);
    // (readlane returns int: widen through uint32_t, not by sign)
    auto at = [&](int w, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)c[w], l); };
    BccDraws d;
    for (int a = 0; a < 3; ++a) d.shift[a] = at(a, 0);
    d.yz_lo = (uint64_t)at(0, 1) | (uint64_t)at(1, 1) << 32;
    d.yz_hi = (uint64_t)at(2, 1) | (uint64_t)at(3, 1) << 32;
    d.x = (uint64_t)at(0, 2) | (uint64_t)at(1, 2) << 32;
    return d;
}

// SLAB: the lattice is a z-slab (DevLattice::slab).
template <bool SLAB>
__device__ __forceinline__ BccBlock bcc_block(const DevLattice& D, int f, int colour, const BccDraws& draws)
{
    BccBlock b;
    // block coordinates: same-colour blocks are every other block per axis
    const int hx = D.nb[0] >> 1, hy = D.nb[1] >> 1;
    const int kx = 2 * (f % hx) + (colour & 1);
    const int ky = 2 * ((f / hx) % hy) + ((colour >> 1) & 1);
    const int kz = 2 * (f / (hx * hy)) + ((colour >> 2) & 1);
    b.Lx = D.L[0];
    b.Ly = D.L[1];
    b.Lz = D.L[2];

    // origin shift of sweep s (same for every wave of the sweep)
    const int ox = (int)(((uint64_t)draws.shift[0] * (uint32_t)b.Lx) >> 32);
    const int oy = (int)(((uint64_t)draws.shift[1] * (uint32_t)b.Ly) >> 32);
    // a z-slab keeps its blocks aligned to its boundaries: no z shift
    const int oz = SLAB ? 0 : (int)(((uint64_t)draws.shift[2] * (uint32_t)b.Lz) >> 32);

    const int x0 = block_lo(kx, b.Lx, D.nb[0]);
    const int y0 = block_lo(ky, b.Ly, D.nb[1]);
    const int z0 = block_lo(kz, b.Lz, D.nb[2]);
    b.wx = block_lo(kx + 1, b.Lx, D.nb[0]) - x0;
    b.wy = block_lo(ky + 1, b.Ly, D.nb[1]) - y0;
    b.wz = block_lo(kz + 1, b.Lz, D.nb[2]) - z0;
    b.gx0 = wrap_add(x0 + ox, b.Lx);
    b.gy0 = wrap_add(y0 + oy, b.Ly);
    b.gz0 = wrap_add(z0 + oz, b.Lz);
    b.g = D.species;

    b.LxLy = (uint32_t)b.Lx * (uint32_t)b.Ly;
    const uint64_t zspan = SLAB ? (uint64_t)b.Lz + 4 + D.z_off : (uint64_t)b.Lz;
    b.narrow = b.LxLy < (1u << 24) && (uint64_t)b.LxLy * zspan < (1ull << 32);
    b.plane_bytes = 2ull * b.LxLy;
    b.buf_bytes = b.plane_bytes * (uint64_t)(SLAB ? b.Lz + 4 : b.Lz);
    b.plane32 = b.plane_bytes < (1ull << 31);
    return b;
}

// Random-number cell id of the lane's class-0 cell (3 ix, 3 iy, 3 iz) of the
// block; a slab's cells are numbered globally (z_off).
template <bool SLAB>
__device__ __forceinline__ void bcc_base_cell(const BccBlock& B, uint32_t z_off, int ix, int iy, int iz, uint32_t& lo,
                                              uint32_t& hi)
{
    // a lane that holds a site has gx0 + 3 ix < 2 Lx: one conditional
    // subtraction wraps it (other lanes only feed their draws to no trial)
    uint32_t bx = (uint32_t)(B.gx0 + 3 * ix), by = (uint32_t)(B.gy0 + 3 * iy), bz = (uint32_t)(B.gz0 + 3 * iz);
    bx = min(bx, bx - (uint32_t)B.Lx);
    by = min(by, by - (uint32_t)B.Ly);
    bz = SLAB ? bz + z_off : min(bz, bz - (uint32_t)B.Lz);
    const uint64_t cell = B.narrow ? (uint64_t)(__umul24(bz, B.LxLy) + __umul24(by, (uint32_t)B.Lx) + bx)
                                   : ((uint64_t)bz * (uint32_t)B.Ly + by) * (uint32_t)B.Lx + bx;
    lo = (uint32_t)cell;
    hi = (uint32_t)(cell >> 32);
}

// Stage block + halo, HBM -> LDS codes (NW waves share the planes: wave w
// takes planes -2 + w * 16 / NW onwards).  dot_codes: this lattice's rows of
// weights are in the byte-dot form.  `between` (work that needs no loaded
// byte) runs while the loads are in flight.
// (The launches that share a block have planes far below 2 GiB.)
template <int KMAX, class LY, bool SLAB, int NW, class Fn>
__device__ __forceinline__ void bcc_stage(const BccBlock& B, uint8_t* lat, int lane, int w, bool dot_codes, Fn&& between)
{
    static_assert(NW == 1 || NW == 4, "waves per block");
    constexpr int F = Field<KMAX>::F;
    // Rows a lane has in flight at once (registers bound it: two words per row).
    constexpr int ROWS = NW == 1 ? kStageRows : 32 / NW;
    const int lz_first = w * (16 / NW) - 2;
    // species bytes -> LDS codes for this lattice's form of the weight rows
    auto encode = [&](uint32_t v) -> uint32_t {
        if constexpr (KMAX <= 5) {
            if (dot_codes) return encode4_dot<KMAX>(v);
        }
        return encode4(v, F);
    };
    // The same map as a byte table for v_perm_b32, code_hi:code_lo = codes
    // of species 7..0 (species >= KMAX never occur: table byte 0).
    uint32_t code_lo = 0u, code_hi = 0u;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        const uint32_t c = v < KMAX ? encode((uint32_t)v) & 0xffu : 0u;
        if (v < 4) code_lo |= c << (8 * v);
        else code_hi |= c << (8 * (v - 4));
    }
    // v_perm_b32 reads at most one scalar operand: hold one word in a vector
    // register for the whole staging rather than copying it there per row
    asm volatile("" : "+v"(code_lo));

    // Cells lx0, lx0 + 1 of the lane's rows (codes corner, body, corner, body
    // in a word) into the image: row it is row h = it & 1 of plane lz0 + it / 2,
    // corner(lx0, ly, -1) at cl[h] less a plane.  Each of the four bytes has a
    // lane mask of its own, set once for all planes.
    auto put = [&](int lz0, const uint32_t (&v)[ROWS], const int (&cl)[2], const bool (&mc0)[2], const bool (&mc1)[2],
                   const bool (&mb0)[2], const bool (&mb1)[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint8_t* p0 = lat + cl[h] + (lz0 + 1) * LY::PP;      // corner(lx0, ly, lz0)
            uint8_t* q0 = p0 + LY::kBodyFromCorner;
            auto planes = [&](uint8_t* at, int shift, bool body) {
#pragma unroll
                for (int k = 0; k < ROWS / 2; ++k)
                    if (body ? lz0 + k <= 12 : lz0 + k >= -1)   // (wave-uniform)
                        at[k * LY::PP] = (uint8_t)(v[2 * k + h] >> shift);
            };
            if (mc0[h]) planes(p0, 0, false);
            if (mc1[h]) planes(p0 + 1, 16, false);
            if (mb0[h]) planes(q0, 8, true);
            if (mb1[h]) planes(q0 + 1, 24, true);
        }
    };

    // ---- stage block + halo: local cells -2..w+1 on each axis ----
    // Fast path (the block's x-range does not cross the periodic boundary):
    // 8 lanes per row, each taking cells lx0, lx0 + 1 (lx0 = 2 (lane & 7) - 2),
    // i.e. the bytes corner, body, corner, body at byte `at` of the row; it
    // loads the aligned dwords at `at & ~3` and 4 bytes on and aligns them.
    // Lane row lr = lane >> 3 takes rows ly = lr - 2 + 8 h (h = 0, 1) of each
    // plane lz = -2 .. 13.  Per lane, the in-plane byte offsets and LDS
    // positions of its two rows are set up once; a row adds only its plane,
    // which is wave-uniform (the buffer resource's base, scalar registers).
    // All its loads are issued before any LDS write.  Rows, planes
    // and cells past the halo (w < 12) load an in-range cell and write it to
    // image positions past w + 1, which no trial with a site and no
    // write-back reads; only positions outside the 15^3 arrays (corner -2,
    // body 13) are not written.  Every load stays inside the row's plane.
    // (NW = 4 has as many loads in flight either way and takes the second
    // path for every block: one copy of the code.)
    if (NW == 1 && B.plane32 && B.gx0 >= 3 && B.gx0 + B.wx + 4 <= B.Lx) {
        const int c8 = lane & 7, lr = lane >> 3;
        const int lx0 = 2 * c8 - 2;
        const int lxa = lx0 <= B.wx + 1 ? lx0 : -2;   // cells the lane loads
        uint32_t yoff[2];
        int cl[2];
        bool mc0[2], mc1[2], mb0[2], mb1[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ly = lr - 2 + 8 * h;
            const uint32_t gy = (uint32_t)wrap_add(B.gy0 + min(ly, B.wy + 1), B.Ly);
            yoff[h] = 2u * (gy * (uint32_t)B.Lx + (uint32_t)(B.gx0 + lxa));
            cl[h] = (ly + 1) * LY::P + (lx0 + 1);      // corner(lx0, ly, -1), less a plane
            mc0[h] = ly >= -1 && c8 >= 1;
            mc1[h] = ly >= -1;
            mb0[h] = ly <= 12;
            mb1[h] = ly <= 12 && c8 <= 6;
        }
#pragma unroll
        for (int n = 0; n < 32 / NW / ROWS; ++n) {
            const int lz0 = lz_first + n * (ROWS / 2);
            uint32_t v[ROWS];
#pragma unroll
            for (int it = 0; it < ROWS; ++it) {
                const int h = it & 1, lz = lz0 + (it >> 1);
                const uint64_t zb = B.plane_bytes * (uint32_t)B.zplane<SLAB>(min(lz, B.wz + 1));
                const uint64_t base = zb & ~(uint64_t)3;
                const __amdgpu_buffer_rsrc_t r = byte_rsrc(B.g + base, B.buf_bytes - base);
                const uint32_t at = yoff[h] + ((uint32_t)zb & 2u);
                const uint32_t A = at & ~3u;
                v[it] = __builtin_amdgcn_perm(code_hi, code_lo,
                                              __builtin_amdgcn_alignbyte(bload32(r, A + 4), bload32(r, A), at));
            }
            if (n == 0) between();
            put(lz0, v, cl, mc0, mc1, mb0, mb1);
        }
    } else if (NW > 1 || B.plane32) {
        // The x-range crosses the periodic boundary: the rows and LDS
        // positions of the fast path, but each lane loads its two cells
        // separately, one 16-bit load each at its own wrapped x, so that a
        // pair may straddle the boundary.  The plane's byte remainder
        // (zb & 2) goes into the scalar offset of both loads.
        const int c8 = lane & 7, lr = lane >> 3;
        const int lx0 = 2 * c8 - 2;
        const int lxa = lx0 <= B.wx + 1 ? lx0 : -2;   // cells the lane loads
        // gx0 + lxa + 1 <= (Lx - 1) + (wx + 2) < 2 Lx, as wx + 2 <= Lx
        const uint32_t gxa = (uint32_t)wrap_add(B.gx0 + lxa, B.Lx), gxb = (uint32_t)wrap_add(B.gx0 + lxa + 1, B.Lx);
        uint32_t oa[2], ob[2];
        int cl[2];
        bool mc0[2], mc1[2], mb0[2], mb1[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ly = lr - 2 + 8 * h;
            const uint32_t row = (uint32_t)wrap_add(B.gy0 + min(ly, B.wy + 1), B.Ly) * (uint32_t)B.Lx;
            oa[h] = 2u * (row + gxa);
            ob[h] = 2u * (row + gxb);
            cl[h] = (ly + 1) * LY::P + (lx0 + 1);
            mc0[h] = ly >= -1 && c8 >= 1;
            mc1[h] = ly >= -1;
            mb0[h] = ly <= 12;
            mb1[h] = ly <= 12 && c8 <= 6;
        }
#pragma unroll
        for (int n = 0; n < 32 / NW / ROWS; ++n) {
            const int lz0 = lz_first + n * (ROWS / 2);
            uint32_t v[ROWS], v2[ROWS];
#pragma unroll
            for (int it = 0; it < ROWS; ++it) {
                const int h = it & 1, lz = lz0 + (it >> 1);
                const uint64_t zb = B.plane_bytes * (uint32_t)B.zplane<SLAB>(min(lz, B.wz + 1));
                const uint64_t base = zb & ~(uint64_t)3;
                const __amdgpu_buffer_rsrc_t r = byte_rsrc(B.g + base, B.buf_bytes - base);
                const int so = (int)((uint32_t)zb & 2u);
                v[it] = __builtin_amdgcn_raw_buffer_load_b16(r, (int)oa[h], so, 0);
                v2[it] = __builtin_amdgcn_raw_buffer_load_b16(r, (int)ob[h], so, 0);
            }
            if (n == 0) {
                __builtin_amdgcn_sched_barrier(0);
                between();
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int it = 0; it < ROWS; ++it) v[it] = __builtin_amdgcn_perm(code_hi, code_lo, v[it] | v2[it] << 16);
            put(lz0, v, cl, mc0, mc1, mb0, mb1);
        }
    } else if constexpr (NW == 1) {
        // planes of 2 GiB or more: one cell (two bytes) per lane, rows
        // r = (lane >> 4) + 4 it, 64-bit addresses; all 64 loads of a lane
        // are issued before any LDS write, as on the fast path (lanes and
        // rows outside the halo load a clamped in-range cell)
        between();
        constexpr int BATCH = 16;
        const int lx = (lane & 15) - 2;
        const bool okx = lx <= B.wx + 1;
        const int gx = wrap_add(B.gx0 + (okx ? lx : -2), B.Lx);
#pragma unroll
        for (int it0 = 0; it0 < 64; it0 += 2 * BATCH) {
            uint32_t v2[2 * BATCH];
#pragma unroll
            for (int u = 0; u < 2 * BATCH; ++u) {
                const int it = it0 + u;
                const int ly = min((lane >> 4) + 4 * (it & 3) - 2, B.wy + 1), lz = min((it >> 2) - 2, B.wz + 1);
                const int gy = wrap_add(B.gy0 + ly, B.Ly);
                const size_t cell = ((size_t)B.zplane<SLAB>(lz) * B.Ly + gy) * B.Lx + gx;
                v2[u] = gload<uint16_t>(B.g + 2 * cell);
            }
#pragma unroll
            for (int u = 0; u < 2 * BATCH; ++u) {
                const int it = it0 + u;
                const int ly = (lane >> 4) + 4 * (it & 3) - 2, lz = (it >> 2) - 2;
                if (!okx || ly > B.wy + 1 || lz > B.wz + 1) continue;
                const uint32_t v = encode(v2[u]);
                if (lx >= -1 && ly >= -1 && lz >= -1)
                    lat[(lz + 1) * LY::PP + (ly + 1) * LY::P + (lx + 1)] = (uint8_t)v;
                if (lx <= B.wx && ly <= B.wy && lz <= B.wz)
                    lat[LY::ARR + (lz + 2) * LY::PP + (ly + 2) * LY::P + (lx + 2)] = (uint8_t)(v >> 8);
            }
        }
    }
}

// Write the block and its first-neighbour ring back (wave w takes every
// NW-th pair of planes).
template <class LY, bool SLAB, int NW>
__device__ __forceinline__ void bcc_write_back(const BccBlock& B, const uint8_t* lat, int lane, int w)
{
    // ---- write back ----
    // A trial changes only corner cells 0..w and body cells -1..w-1 of the
    // block (its sites and their first neighbours).  Row path (planes under
    // 2 GiB): every cell of the box -1..w on each axis is written
    // whole (corner and body byte, one 16-bit store), the cells no trial
    // could change with the value staged from them.  That is the value they
    // still hold: no block of the same colour changes them (same-colour
    // blocks are one block of width >= 2 apart along some axis, and their
    // changes reach one cell beyond their own cells), and the cells of the
    // box are distinct (L >= w + 2 on each axis: at least 2 blocks of width
    // >= 2).  16 lanes per row (lx = (lane & 15) - 1) and 4 rows per
    // instruction: lane row lys = lane >> 4 takes rows ly = 4 yg + lys - 1
    // (yg = 0..3) of each plane lz = -1..w.  Per lane, the in-plane byte
    // offsets and LDS positions of its four rows are set up once; lanes past
    // the box read a clamped in-image cell and store past the plane, which the
    // resource's bound drops.  A lane's x is
    // wrapped once here, so blocks whose x-range crosses the periodic
    // boundary take this path too (same-colour blocks are as far apart
    // across the boundary as anywhere else, nb being even).
    if (NW > 1 || B.plane32) {
        const int lx = (lane & 15) - 1, lys = lane >> 4;
        const int lxc = min(lx, B.wx);
        uint32_t yo[4];
        int cw[4];
#pragma unroll
        for (int yg = 0; yg < 4; ++yg) {
            const int ly = 4 * yg + lys - 1, lyc = min(ly, B.wy);
            const uint32_t gy = (uint32_t)wrap_add(B.gy0 + lyc, B.Ly);
            const uint32_t at = 2u * (gy * (uint32_t)B.Lx + (uint32_t)wrap_add(B.gx0 + lxc, B.Lx));
            yo[yg] = lx <= B.wx && ly <= B.wy ? at : 1u << 31;   // past the plane: the store is dropped
            cw[yg] = (lyc + 1) * LY::P + (lxc + 1);   // corner(lxc, lyc, -1), less a plane
        }
        // two planes at a time: their LDS reads are issued together (the
        // second of an odd last pair is the first again)
        constexpr int PAIRS = (kMaxBlock + 2 + 2 * NW - 1) / (2 * NW);
#pragma unroll
        for (int k = 0; k < PAIRS; ++k) {
            const int lz0 = 2 * (NW * k + w) - 1;
            if (lz0 > B.wz) continue;   // (wave-uniform)
            uint32_t e[2][4];
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int yg = 0; yg < 4; ++yg) {
                    const uint8_t* p = lat + cw[yg] + (min(lz0 + n, B.wz) + 1) * LY::PP;   // corner(lxc, lyc, lz)
                    e[n][yg] = (uint32_t)p[0] | (uint32_t)p[LY::kBodyFromCorner] << 8;
                }
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const uint64_t zb = B.plane_bytes * (uint32_t)B.zplane<SLAB>(min(lz0 + n, B.wz));
                const __amdgpu_buffer_rsrc_t r = byte_rsrc(B.g + zb, B.plane_bytes);
#pragma unroll
                for (int yg = 0; yg < 4; ++yg) bstore16(r, yo[yg], (e[n][yg] >> 5) & 0x0707u);
            }
        }
    } else if constexpr (NW == 1) {
        // planes of 2 GiB or more: one cell (two bytes) per lane, rows
        // r = (lane >> 4) + 4 it, 64-bit addresses; the LDS reads of 8 rows
        // are issued together (rows and cells outside the boxes read clamped in-image
        // bytes and store nothing)
        const int lx = (lane & 15) - 1;
        const bool okx = lx <= B.wx;
        const int lxc = okx ? lx : B.wx;
        const int gx = wrap_add(B.gx0 + lxc, B.Lx);
        const int nit = 4 * (B.wz + 2);               // rows with lz <= B.wz
        for (int it0 = 0; it0 < nit; it0 += 8) {
            uint32_t vc[8], vb[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int it = it0 + u;
                const int lyc = min((lane >> 4) + 4 * (it & 3) - 1, B.wy), lzc = min((it >> 2) - 1, B.wz);
                vc[u] = lat[(lzc + 1) * LY::PP + (lyc + 1) * LY::P + (lxc + 1)];
                vb[u] = lat[LY::ARR + (lzc + 2) * LY::PP + (lyc + 2) * LY::P + (lxc + 2)];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int it = it0 + u;
                const int ly = (lane >> 4) + 4 * (it & 3) - 1, lz = (it >> 2) - 1;
                if (!okx || ly > B.wy || lz > B.wz) continue;
                const bool corner = lx >= 0 && ly >= 0 && lz >= 0;
                const bool body = lx < B.wx && ly < B.wy && lz < B.wz;
                if (!corner && !body) continue;
                const int gy = wrap_add(B.gy0 + ly, B.Ly);
                const size_t cell = ((size_t)B.zplane<SLAB>(lz) * B.Ly + gy) * B.Lx + gx;
                if (corner && body)
                    gstore<uint16_t>(B.g + 2 * cell, (uint16_t)(decode(vc[u]) | decode(vb[u]) << 8));
                else if (corner)
                    gstore<uint8_t>(B.g + 2 * cell, (uint8_t)decode(vc[u]));
                else
                    gstore<uint8_t>(B.g + 2 * cell + 1, (uint8_t)decode(vb[u]));
            }
        }
    }
}

}  // namespace smcx
