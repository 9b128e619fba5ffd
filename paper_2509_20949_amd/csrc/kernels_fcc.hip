// kernels_fcc.hip -- the sweep kernel on the FCC lattice
// (the lattice of the paper's quinary alloy and its L1_2 precipitates).
//
// Four sublattices per cubic cell at doubled offsets SUB[b]; 12/6/24
// neighbours in shells 1/2/3.  One wavefront per block as on BCC; the LDS
// image holds one 15^3 byte array per sublattice, array b covering local
// cells -1-SUB[b][a] .. 13-SUB[b][a] along axis a, so every neighbour offset
// is a compile-time constant for a given (sublattice, displacement).  A
// round is one (residue class, sublattice) pair: 27 x 4 = 108 rounds.
//
// Partner choice: the partner of all trials of one (sweep, colour,
// sub-colour) set -- its sublattice and the signs of the step on the two
// axes where the sublattices differ -- is drawn once (the same draw on
// every wave), so a scalar branch selects a trial specialised on it, which
// reads only the cells its energy change needs (the symmetric difference of
// the site's and the partner's shells), every read of a wave at one common
// offset.  A trial's own draw is its acceptance word: one Philox call per
// cell serves the cell's four sites.  (The FCC pair counts are in
// pair_counts.hip.)
#include <type_traits>

#include "device_common.h"

namespace smcx {
namespace fcc {

constexpr int SUB[4][3] = {{0, 0, 0}, {1, 1, 0}, {1, 0, 1}, {0, 1, 1}};
constexpr int SH1[12][3] = {{+1, +1, 0}, {+1, -1, 0}, {-1, +1, 0}, {-1, -1, 0}, {+1, 0, +1}, {+1, 0, -1},
                            {-1, 0, +1}, {-1, 0, -1}, {0, +1, +1}, {0, +1, -1}, {0, -1, +1}, {0, -1, -1}};
constexpr int SH2[6][3] = {{+2, 0, 0}, {-2, 0, 0}, {0, +2, 0}, {0, -2, 0}, {0, 0, +2}, {0, 0, -2}};
constexpr int SH3[24][3] = {{+2, +1, +1}, {+2, +1, -1}, {+2, -1, +1}, {+2, -1, -1}, {-2, +1, +1}, {-2, +1, -1},
                            {-2, -1, +1}, {-2, -1, -1}, {+1, +2, +1}, {+1, +2, -1}, {-1, +2, +1}, {-1, +2, -1},
                            {+1, -2, +1}, {+1, -2, -1}, {-1, -2, +1}, {-1, -2, -1}, {+1, +1, +2}, {+1, -1, +2},
                            {-1, +1, +2}, {-1, -1, +2}, {+1, +1, -2}, {+1, -1, -2}, {-1, +1, -2}, {-1, -1, -2}};
constexpr int kArrays = 4;
constexpr int kWaveLdsF = kArrays * kArr;

constexpr int origin(int b, int a) { return 1 + SUB[b][a]; }
constexpr int stride(int a) { return a == 0 ? 1 : (a == 1 ? kP : kPP); }
constexpr int sub_of_parity(int px, int py, int pz)
{
    return (px == 0 && py == 0 && pz == 0) ? 0 : (px && py && !pz) ? 1 : (px && !py && pz) ? 2 : 3;
}
constexpr int fdiv2(int t) { return t >= 0 ? t / 2 : -((-t + 1) / 2); }
constexpr int mod2(int t) { return t & 1; }

// LDS offset from the site (b, cell) to the site at doubled displacement d.
constexpr int offset(int b, int dx, int dy, int dz)
{
    const int d[3] = {dx, dy, dz};
    int par[3] = {0, 0, 0}, cd[3] = {0, 0, 0};
    for (int a = 0; a < 3; ++a) {
        const int t = SUB[b][a] + d[a];
        par[a] = mod2(t);
        cd[a] = fdiv2(t);
    }
    const int bp = sub_of_parity(par[0], par[1], par[2]);
    int off = (bp - b) * kArr;
    for (int a = 0; a < 3; ++a) off += (cd[a] + origin(bp, a) - origin(b, a)) * stride(a);
    return off;
}

// The two axes on which sublattices B and BP differ.
constexpr int axis1(int B, int BP) { return SUB[B][0] != SUB[BP][0] ? 0 : 1; }
constexpr int axis2(int B, int BP) { return SUB[B][2] != SUB[BP][2] ? 2 : 1; }

// The cells a trial must load, for the site in sublattice B and its partner
// in sublattice BP with signs SG (bit 0: first differing axis, bit 1:
// second; set = +1), counting shells s < S.  In doubled coordinates the
// partner is at dj, and what the energy change needs per shell s is
// sum over N_s of e(i + v) - sum over N_s of e(i + dj + v): cells in both
// N_s(i) and N_s(j) cancel.  The rest, the symmetric differences, are 50
// distinct cells for S = 3 (against 2 x 42 neighbours), some counted in two
// shells.  plus/minus: bit s set = +1 / -1 in shell s.  The partner (dj, in
// i's first shell) and the site itself (in j's first shell) are among them.
struct DiffCells {
    int n;
    int off[64];
    int plus[64], minus[64];
    int i_site, i_partner;   // indices of the site and of the partner
    int off_partner;         // LDS offset of the partner
};

constexpr int find_cell(const int (&d)[64][3], int n, int x, int y, int z)
{
    for (int k = 0; k < n; ++k)
        if (d[k][0] == x && d[k][1] == y && d[k][2] == z) return k;
    return -1;
}

constexpr bool in_shell(int s, int x, int y, int z)
{
    const int r = x * x + y * y + z * z;
    return ((x + y + z) & 1) == 0 && r == (s == 0 ? 2 : s == 1 ? 4 : 6);
}

constexpr DiffCells make_diff(int B, int BP, int SG, int S)
{
    DiffCells c{};
    int d[64][3] = {};
    int dj[3] = {0, 0, 0};
    dj[axis1(B, BP)] = (SG & 1) ? 1 : -1;
    dj[axis2(B, BP)] = (SG & 2) ? 1 : -1;
    for (int s = 0; s < S; ++s) {
        const int n = s == 0 ? 12 : s == 1 ? 6 : 24;
        for (int k = 0; k < n; ++k) {
            const int* v = s == 0 ? SH1[k] : s == 1 ? SH2[k] : SH3[k];
            // i's neighbour v, unless it is also j's neighbour in shell s
            if (!in_shell(s, v[0] - dj[0], v[1] - dj[1], v[2] - dj[2])) {
                int t = find_cell(d, c.n, v[0], v[1], v[2]);
                if (t < 0) { t = c.n++; d[t][0] = v[0]; d[t][1] = v[1]; d[t][2] = v[2]; }
                c.plus[t] |= 1 << s;
            }
            // j's neighbour dj + v, unless it is also i's neighbour in shell s
            const int w0 = dj[0] + v[0], w1 = dj[1] + v[1], w2 = dj[2] + v[2];
            if (!in_shell(s, w0, w1, w2)) {
                int t = find_cell(d, c.n, w0, w1, w2);
                if (t < 0) { t = c.n++; d[t][0] = w0; d[t][1] = w1; d[t][2] = w2; }
                c.minus[t] |= 1 << s;
            }
        }
    }
    for (int k = 0; k < c.n; ++k) c.off[k] = offset(B, d[k][0], d[k][1], d[k][2]);
    c.i_site = find_cell(d, c.n, 0, 0, 0);
    c.i_partner = find_cell(d, c.n, dj[0], dj[1], dj[2]);
    c.off_partner = offset(B, dj[0], dj[1], dj[2]);
    return c;
}

template <int B, int BP, int SG, int S> struct Diff { static constexpr DiffCells v = make_diff(B, BP, SG, S); };

// Species fields: 6 bits each (up to 24 neighbours per shell), 5 species,
// biased by 32 so that 32 + n_i - n_j never borrows.
constexpr int F = 6;
constexpr int KMAXF = 5;
constexpr uint32_t kBias = 32u * (1u | 1u << 6 | 1u << 12 | 1u << 18 | 1u << 24);

// The cells of a trial in the order it counts them: those that count in shell
// s with sign + or - as lists of cell indices, and the loads that no earlier
// list has asked for.
struct CountLists {
    int n[kMaxS][2];
    int cell[kMaxS][2][32];
    int n_load;
    int load[64];   // cells in load order: site, partner, then as counted
};
template <int S> constexpr CountLists make_lists(const DiffCells& c)
{
    CountLists l{};
    bool seen[64] = {};
    l.load[l.n_load++] = c.i_site;
    l.load[l.n_load++] = c.i_partner;
    seen[c.i_site] = seen[c.i_partner] = true;
    for (int s = 0; s < S; ++s)
        for (int sign = 0; sign < 2; ++sign)
            for (int k = 0; k < c.n; ++k)
                if ((sign ? c.minus[k] : c.plus[k]) >> s & 1) {
                    l.cell[s][sign][l.n[s][sign]++] = k;
                    if (!seen[k]) {
                        seen[k] = true;
                        l.load[l.n_load++] = k;
                    }
                }
    return l;
}
template <int B, int BP, int SG, int S> struct Lists {
    static constexpr DiffCells cells = Diff<B, BP, SG, S>::v;
    static constexpr CountLists v = make_lists<S>(cells);
};

// Loads From .. To - 1 of the load order into c.
template <class L, int From, int To>
__device__ __forceinline__ void load_cells(uint32_t (&c)[64], const uint8_t* lat, int ai)
{
    if constexpr (From < To) {
        constexpr int k = L::v.load[From], off = L::cells.off[k];
        c[k] = lat[ai + off];
        load_cells<L, From + 1, To>(c, lat, ai);
    }
}

// Counts entries At .. of list (s, sign) into h, four to an asm block.
template <class L, int s, int sign, int At = 0>
__device__ __forceinline__ void count_list(uint32_t& h, const uint32_t (&c)[64])
{
    constexpr int left = L::v.n[s][sign] - At;
    if constexpr (left > 0) {
        constexpr const int* list = L::v.cell[s][sign];
        constexpr int k0 = list[At], k1 = list[At + (left > 1)], k2 = list[At + 2 * (left > 2)],
                      k3 = list[At + 3 * (left > 3)];
        if constexpr (left >= 4) {
            count4<sign == 1>(h, c[k0], c[k1], c[k2], c[k3]);
            count_list<L, s, sign, At + 4>(h, c);
        } else if constexpr (left == 3) {
            count3<sign == 1>(h, c[k0], c[k1], c[k2]);
        } else if constexpr (left == 2) {
            count2<sign == 1>(h, c[k0], c[k1]);
        } else {
            count1<sign == 1>(h, c[k0]);
        }
    }
}

// One trial: site at LDS byte ai (sublattice B), partner in sublattice BP
// with the signs SG (bit 0: first differing axis, bit 1: second; set = +1),
// all three wave-uniform, acceptance draw u.  MODE: the form of the weight
// rows (per lattice): kWtabDot or kWtabFull.
// The site's and the partner's codes are loaded first, so that their weight
// row is requested while the other cells are still arriving; every load is
// issued before the first count.
template <int SMAX, int MODE, int B, int BP, int SG>
__device__ __forceinline__ void trial(uint8_t* lat, int ai, uint32_t u, uint64_t valid, const int32_t* wtab,
                                      const double* tab, float ln2kT, Sums& sums)
{
    constexpr bool DOT = MODE == kWtabDot;
    using L = Lists<B, BP, SG, SMAX>;
    constexpr DiffCells C = L::cells;
    static_assert(C.n <= 64 && C.i_site >= 0 && C.i_partner >= 0 && L::v.n_load == C.n, "cell table");
    constexpr int kAhead = C.n < 14 ? C.n : 14;   // (the LDS counter tells at most 15 loads in flight apart)
    uint32_t c[64];
    load_cells<L, 0, kAhead>(c, lat, ai);
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t ci = c[C.i_site], cj = c[C.i_partner];
    // row (a, b) of the weight planes at byte 4 (5 a + b) of a plane
    const uint32_t row4 = __umul24(ci >> 5, 4u * KMAXF) + ((cj >> 5) << 2);
    const int32_t* w = (const int32_t*)((const uint8_t*)wtab + row4);
    constexpr int NW = DOT ? 3 * SMAX + 1 : 1;
    int32_t row[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) row[k] = w[(DOT ? k : SMAX * KMAXF) * kPlane];
    load_cells<L, kAhead, C.n>(c, lat, ai);
    __builtin_amdgcn_sched_barrier(0);
    const Edges edges = edges_of(u, ln2kT);   // depends on the draw only
    // packed per-shell fields bias + n_i - n_j over the symmetric
    // differences (6-bit fields, or bytes in the byte-dot form)
    uint32_t h[kMaxS];
#pragma unroll
    for (int s = 0; s < kMaxS; ++s) h[s] = DOT ? 0x20202020u : kBias;
    count_list<L, 0, 0>(h[0], c);
    count_list<L, 0, 1>(h[0], c);
    if constexpr (SMAX >= 2) {
        count_list<L, 1, 0>(h[1], c);
        count_list<L, 1, 1>(h[1], c);
    }
    if constexpr (SMAX >= 3) {
        count_list<L, 2, 0>(h[2], c);
        count_list<L, 2, 1>(h[2], c);
    }
    uint32_t acc;
    if constexpr (DOT) {
        // bytes 32 + n_i - n_j (bit 31, the last species, masked off) dotted
        // with the three base-256 digits of the folded weights, in one
        // chain: ((A2 * 256 + A1) * 256 + constant) + A0
        int32_t dd[kMaxS];
#pragma unroll
        for (int s = 0; s < SMAX; ++s) dd[s] = (int32_t)(h[s] & 0x7fffffffu);
        int32_t X = 0;
#pragma unroll
        for (int s = 0; s < SMAX; ++s) X = __builtin_amdgcn_sdot4(dd[s], row[3 * s + 2], X, false);
        X = (int32_t)((uint32_t)X << 8);
#pragma unroll
        for (int s = 0; s < SMAX; ++s) X = __builtin_amdgcn_sdot4(dd[s], row[3 * s + 1], X, false);
        X = (int32_t)(((uint32_t)X << 8) + (uint32_t)row[3 * SMAX]);
#pragma unroll
        for (int s = 0; s < SMAX; ++s) X = __builtin_amdgcn_sdot4(dd[s], row[3 * s], X, false);
        acc = (uint32_t)X;
    } else {
        acc = (uint32_t)row[0];
#pragma unroll
        for (int s = 0; s < SMAX; ++s) {
#pragma unroll
            for (int p = 0; p < KMAXF; ++p) acc = mad24((h[s] >> (F * p)) & 63u, w[(s * KMAXF + p) * kPlane], acc);
        }
    }
    const int32_t dE = (int32_t)acc;
    const uint64_t ok = accepted_lanes(dE, u, edges, valid, tab);
    // both bytes stored by every lane (unchanged unless accepted): no two
    // lanes of a round touch the same byte
    const bool accept = __builtin_amdgcn_inverse_ballot_w64(ok);
    lat[ai] = (uint8_t)(accept ? cj : ci);
    lat[ai + C.off_partner] = (uint8_t)(accept ? ci : cj);
    sums.dE += accept ? dE : 0;   // (0 for equal species: their row is zero)
    sums.nacc += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(ci != cj) & ok);
}

// The trial of one of twelve partners (wave-uniform: index k of the partner
// sublattice among those other than B in bits 2 and 3, signs in bits 0 and 1).
// Tests of k, then of the signs, one after the other, each a compare and a
// branch over the code it guards: as a switch the compiler makes every level
// of the tree a chain of flags and branches (21 branches and 65 scalar
// instructions a trial).  The empty asm keeps it from threading the tests
// together again.
template <int SMAX, int MODE, int B, int K>
__device__ __forceinline__ void trial_signs(int p, uint8_t* lat, int ai, uint32_t u, uint64_t valid,
                                            const int32_t* wtab, const double* tab, float ln2kT, Sums& sums)
{
    constexpr int BP = K + (K >= B ? 1 : 0);
    if (p == 4 * K) trial<SMAX, MODE, B, BP, 0>(lat, ai, u, valid, wtab, tab, ln2kT, sums);
    asm volatile("" : "+s"(p));
    if (p == 4 * K + 1) trial<SMAX, MODE, B, BP, 1>(lat, ai, u, valid, wtab, tab, ln2kT, sums);
    asm volatile("" : "+s"(p));
    if (p == 4 * K + 2) trial<SMAX, MODE, B, BP, 2>(lat, ai, u, valid, wtab, tab, ln2kT, sums);
    asm volatile("" : "+s"(p));
    if (p == 4 * K + 3) trial<SMAX, MODE, B, BP, 3>(lat, ai, u, valid, wtab, tab, ln2kT, sums);
}
template <int SMAX, int MODE, int B>
__device__ __forceinline__ void trial_any(int p, uint8_t* lat, int ai, uint32_t u, uint64_t valid, const int32_t* wtab,
                                          const double* tab, float ln2kT, Sums& sums)
{
    if (p < 4) trial_signs<SMAX, MODE, B, 0>(p, lat, ai, u, valid, wtab, tab, ln2kT, sums);
    asm volatile("" : "+s"(p));
    if ((p & 12) == 4) trial_signs<SMAX, MODE, B, 1>(p, lat, ai, u, valid, wtab, tab, ln2kT, sums);
    asm volatile("" : "+s"(p));
    if (p >= 8) trial_signs<SMAX, MODE, B, 2>(p, lat, ai, u, valid, wtab, tab, ln2kT, sums);
}

template <int B>
__device__ __forceinline__ int site_addr(int lx, int ly, int lz)
{
    return B * kArr + (lz + origin(B, 2)) * kPP + (ly + origin(B, 1)) * kP + (lx + origin(B, 0));
}

// Site b of cell l is staged when l_a lies in -1-SUB[b][a] .. w_a+1-SUB[b][a]
// and written back when l_a lies in -SUB[b][a] .. w_a-SUB[b][a] (the block's
// own cells and the partners its trials can reach); its byte in the image is
// b*kArr + (lz+1+SUB[b][2])*kPP + (ly+1+SUB[b][1])*kP + (lx+1+SUB[b][0]).

}  // namespace fcc

// WPG waves (blocks) per workgroup: 2 (five workgroups per CU, LDS-bound), or
// kWavesPerGroupFccWide for a single lattice whose colour then fits the chip
// in fewer generations (one workgroup of 11 block images fills a CU's LDS).
// What bounds it (336 x 315 x 315 cells, S = 3, 11 waves on a CU, so three on
// most SIMDs): latency with three waves to hide it, vector issue (0.59 of those
// SIMDs' cycles) and the LDS (busy 0.52); 139 VALU, 63 LDS and 45 scalar
// instructions per wave-round.
// 166 us a launch before the site and partner were loaded first (150), the
// partner's arms stood behind flat tests (143) and staging and write-back were
// set up once per lane (136).
template <int SMAX, int WPG>
__global__ __launch_bounds__(kWave * WPG)
void sweep_phase_fcc_kernel(const DevLattice* __restrict__ lats, const WorkItem* __restrict__ items, int n_groups,
                            int t, int colour)
{
    using namespace fcc;
    // the weight planes at LDS offset 0 (row addresses need no base), then
    // the block images
    constexpr int kWords = wplanes(KMAXF, SMAX) * kPlane, kWPer = (kWords + kWave * WPG - 1) / (kWave * WPG);
    __shared__ __attribute__((aligned(16))) uint8_t s_mem[4 * kWords + WPG * kWaveLdsF];
    int32_t* s_w = (int32_t*)s_mem;
    uint8_t* s_lat = s_mem + 4 * kWords;

    const int wave = wave_id();
    const int lane = threadIdx.x % kWave;
    // group grp of the launch's n_groups (XCD-aware order): work item g of a
    // batched launch, or blocks WPG g .. WPG g + WPG - 1 of a single lattice
    const int grp = xcd_group(n_groups);
    if (grp < 0) return;   // no later barrier in a workgroup without a group
    int li = 0, f = grp * WPG;
    if (items) {
        li = items[grp].lattice;
        f = items[grp].first_block;
    }
    const DevLattice& D = lats[li];
    const uint32_t s = D.sweep0 + (uint32_t)t;
    // the words of the weight planes, on their way while the block is set up;
    // the threshold tables stay in global memory
    int32_t wword[kWPer];
#pragma unroll
    for (int n = 0; n < kWPer; ++n) {
        const int k = n * kWave * WPG + (int)threadIdx.x, row = k % kPlane;
        wword[n] = k < kWords && row < KMAXF * KMAXF ? D.wtab[row * wrow(KMAXF, SMAX) + k / kPlane] : 0;
    }
    int ti = (int)(s - D.tab_s0);
    ti = ti < 0 ? 0 : (ti >= D.n_tabs ? D.n_tabs - 1 : ti);
    const double* g_tab = D.tabs + (size_t)ti * kTab;
    const float ln2kT = (float)g_tab[kTabLn2kT];
    f += wave;
    const bool active = f < D.blocks_per_colour;   // wave-uniform; the group's last waves may have no block
    if (!active) f = 0;

    const int hx = D.nb[0] >> 1, hy = D.nb[1] >> 1;
    const int kx = 2 * (f % hx) + (colour & 1);
    const int ky = 2 * ((f / hx) % hy) + ((colour >> 1) & 1);
    const int kz = 2 * (f / (hx * hy)) + ((colour >> 2) & 1);
    const int Lx = D.L[0], Ly = D.L[1], Lz = D.L[2];
    const uint32_t k0 = D.key[0], k1 = D.key[1];
    // partner of every (colour, sub-colour q) set of this sweep, from
    // r = Philox(key, (q, 0, s, c + 64)): sublattice = the k-th other than
    // the set's own, k = (r0 * 3) >> 32 (bits 2 and 3), signs = bits 30 and 31
    // of r1 (bits 0 and 1).  Lane q (q - 64) of part[0] (part[1]) holds it;
    // the origin shift (0, 0, s, 8) takes an idle lane of the second call.
    int part[2];
    uint32_t sh[3];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int q = 64 * h + lane;
        const bool own_shift = h == 1 && lane == 63;
        uint32_t r[4] = {own_shift ? 0u : (uint32_t)q, 0u, s, own_shift ? 8u : (uint32_t)colour + 64u};
        philox4x32_10(r, k0, k1);
        if (h == 1)
            for (int a = 0; a < 3; ++a) sh[a] = (uint32_t)__builtin_amdgcn_readlane((int)r[a], 63);
        part[h] = (int)(((uint64_t)r[0] * 3u) >> 32) << 2 | (int)(r[1] >> 30);
    }
    const int ox = (int)(((uint64_t)sh[0] * (uint32_t)Lx) >> 32);
    const int oy = (int)(((uint64_t)sh[1] * (uint32_t)Ly) >> 32);
    const int oz = (int)(((uint64_t)sh[2] * (uint32_t)Lz) >> 32);
    const int x0 = block_lo(kx, Lx, D.nb[0]), wx = block_lo(kx + 1, Lx, D.nb[0]) - x0;
    const int y0 = block_lo(ky, Ly, D.nb[1]), wy = block_lo(ky + 1, Ly, D.nb[1]) - y0;
    const int z0 = block_lo(kz, Lz, D.nb[2]), wz = block_lo(kz + 1, Lz, D.nb[2]) - z0;
    const int gx0 = wrap_add(x0 + ox, Lx), gy0 = wrap_add(y0 + oy, Ly), gz0 = wrap_add(z0 + oz, Lz);

    uint8_t* lat = s_lat + wave * kWaveLdsF;
    uint8_t* __restrict__ g = D.species;

    const bool dot_codes = D.drop_last == kWtabDot;   // LDS codes for the byte-dot weight rows
    // ---- stage block + halo: one cell (4 sublattice bytes, one dword) per lane ----
    // Lane row lr = lane >> 4 takes the cells lx = (lane & 15) - 2 of rows
    // ly = lr - 2 + 4 j (j = 0..3) of each plane lz = -2 .. wz + 1.  The lane's
    // four row addresses are set up once; a plane adds its offset, which is
    // wave-uniform.  The loads of kPlanesF planes are issued together.  Lanes
    // and rows past the halo (w < 12) load an in-range cell and write it to
    // image positions past w + 1, which no trial with a site and no write-back
    // reads; only positions outside the 15^3 arrays (-2 or, where the
    // sublattice's origin is half a cell lower, 13) are not written.  The
    // writes of one sublattice share their lane mask: -2 and 13 of x for all,
    // of y in the first or the last of the four rows.
    const int64_t plane_bytes = 4 * (int64_t)Lx * Ly;
    constexpr int kPlanesF = 4;
    if (active) {
        // codes of species 0..7 as a byte table (species >= KMAXF never occur)
        uint32_t code_lo = 0u, code_hi = 0u;
#pragma unroll
        for (uint32_t v = 0; v < KMAXF; ++v) {
            const uint32_t c = (dot_codes ? encode4_dot<KMAXF>(v) : (v << 5) + (v << 2) + (v << 1)) & 0xffu;
            if (v < 4) code_lo |= c << (8 * v);
            else code_hi |= c << (8 * (v - 4));
        }
        asm volatile("" : "+v"(code_lo));   // (v_perm_b32 reads at most one scalar operand)
        const int lr = lane >> 4, lx = (lane & 15) - 2;
        const int gx = wrap_add(gx0 + (lx <= wx + 1 ? lx : -2), Lx);
        const uint8_t* row[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int gy = wrap_add(gy0 + min(lr + 4 * j - 2, wy + 1), Ly);
            row[j] = g + 4 * ((size_t)gy * Lx + gx);
        }
        // cell (-1, -1, -1) of sublattice 0 is byte 0 of the image
        uint8_t* at = lat + (lr - 1) * kP + (lx + 1);
#pragma nounroll
        for (int lz0 = -2; lz0 <= wz + 1; lz0 += kPlanesF) {
            uint32_t v[kPlanesF][4];
#pragma unroll
            for (int k = 0; k < kPlanesF; ++k) {
                const int64_t plane = (int64_t)wrap_add(gz0 + min(lz0 + k, wz + 1), Lz) * plane_bytes;
#pragma unroll
                for (int j = 0; j < 4; ++j) v[k][j] = gload<uint32_t>(row[j] + plane);
            }
#pragma unroll
            for (int k = 0; k < kPlanesF; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) v[k][j] = __builtin_amdgcn_perm(code_hi, code_lo, v[k][j]);
            uint8_t* at0 = at + (lz0 + 1) * kPP;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int sx = SUB[b][0], sy = SUB[b][1], sz = SUB[b][2];
                auto put = [&](int j) {
#pragma unroll
                    for (int k = 0; k < kPlanesF; ++k)
                        if (sz ? lz0 + k <= 12 : lz0 + k >= -1)   // (wave-uniform)
                            at0[b * kArr + (k + sz) * kPP + (4 * j + sy) * kP + sx] = (uint8_t)(v[k][j] >> (8 * b));
                };
                if (sx ? lx <= 12 : lx >= -1) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j != (sy ? 3 : 0)) put(j);
                    if (sy ? lr <= 2 : lr >= 1) put(sy ? 3 : 0);   // (ly <= 12, ly >= -1)
                }
            }
        }
    }

#pragma unroll
    for (int n = 0; n < kWPer; ++n) {
        const int k = n * kWave * WPG + (int)threadIdx.x;
        if (k < kWords) s_w[k] = wword[n];
    }
    __syncthreads();
    if (!active) return;   // no later barrier

    // ---- 27 residue classes x 4 sublattices = 108 rounds ----
    int ix, iy, iz;
    lane_cell(lane, ix, iy, iz);
    const uint32_t bx = (uint32_t)(gx0 + 3 * ix), by = (uint32_t)(gy0 + 3 * iy), bz = (uint32_t)(gz0 + 3 * iz);
    const uint32_t LxLy = (uint32_t)Lx * (uint32_t)Ly;
    const bool narrow = LxLy < (1u << 24) && (uint64_t)LxLy * (uint32_t)Lz < (1ull << 32);
    int64_t dEsum = 0;
    Sums sums = {0, 0u};
    auto all_rounds = [&](auto mode_tag) {
        constexpr int MODE = decltype(mode_tag)::value;
#pragma nounroll
        for (int m = 0; m < 27; ++m) {
            const int rx = m % 3, ry = (m / 3) % 3, rz = m / 9;
            const uint64_t valid =
                __builtin_amdgcn_ballot_w64((3 * ix < wx - rx) & (3 * iy < wy - ry) & (3 * iz < wz - rz));
            uint32_t gx = bx + rx, gy = by + ry, gz = bz + rz;
            gx = min(gx, gx - (uint32_t)Lx);
            gy = min(gy, gy - (uint32_t)Ly);
            gz = min(gz, gz - (uint32_t)Lz);
            uint64_t cell;
            if (narrow)
                cell = __umul24(gz, LxLy) + __umul24(gy, (uint32_t)Lx) + gx;
            else
                cell = ((uint64_t)gz * (uint32_t)Ly + gy) * (uint32_t)Lx + gx;
            // one Philox call per cell: site b accepts with word b
            uint32_t ra[4] = {(uint32_t)cell, (uint32_t)(cell >> 32), s, (uint32_t)colour};
            philox4x32_10(ra, k0, k1);
            const int q0 = 4 * m, pv = q0 < 64 ? part[0] : part[1];   // (readlane takes the lane modulo 64)
            uint8_t* at = lat + ((rz + 3 * iz) * kPP + (ry + 3 * iy) * kP + (rx + 3 * ix));
            trial_any<SMAX, MODE, 0>(__builtin_amdgcn_readlane(pv, q0), at, site_addr<0>(0, 0, 0), ra[0], valid, s_w,
                                     g_tab, ln2kT, sums);
            __builtin_amdgcn_wave_barrier();
            trial_any<SMAX, MODE, 1>(__builtin_amdgcn_readlane(pv, q0 + 1), at, site_addr<1>(0, 0, 0), ra[1], valid, s_w,
                                     g_tab, ln2kT, sums);
            __builtin_amdgcn_wave_barrier();
            dEsum += (int64_t)sums.dE;   // (two changes at a time stay inside 32 bits)
            sums.dE = 0;
            trial_any<SMAX, MODE, 2>(__builtin_amdgcn_readlane(pv, q0 + 2), at, site_addr<2>(0, 0, 0), ra[2], valid, s_w,
                                     g_tab, ln2kT, sums);
            __builtin_amdgcn_wave_barrier();
            trial_any<SMAX, MODE, 3>(__builtin_amdgcn_readlane(pv, q0 + 3), at, site_addr<3>(0, 0, 0), ra[3], valid, s_w,
                                     g_tab, ln2kT, sums);
            __builtin_amdgcn_wave_barrier();
            dEsum += (int64_t)sums.dE;
            sums.dE = 0;
        }
    };
    if (dot_codes)
        all_rounds(std::integral_constant<int, kWtabDot>{});
    else
        all_rounds(std::integral_constant<int, kWtabFull>{});

    // ---- write back: sublattice b over cells -SUB[b][a] .. w_a - SUB[b][a] ----
    // Lane row lr takes the cells lx = (lane & 15) - 1 of rows ly = lr - 1 + 4 j
    // of each plane lz = -1 .. wz; the 16 LDS reads of a plane are issued
    // together (lanes and rows outside the boxes read clamped in-image bytes
    // and store nothing).  Cells with all four sublattices in their boxes,
    // 0 .. w_a - 1 on each axis, are stored as a word; of the cells around
    // them each sublattice's own byte.
    {
        const int lr = lane >> 4, lx = (lane & 15) - 1;
        const int gx = wrap_add(gx0 + lx, Lx);
        const bool inner_x = lx >= 0 && lx < wx;
        uint8_t* row[4];
        int src[4];
        bool inner[4], box[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ly = lr + 4 * j - 1;
            row[j] = g + 4 * ((size_t)wrap_add(gy0 + min(ly, wy), Ly) * Lx + gx);
            src[j] = (min(ly, wy) + 1) * kP + (min(lx, wx) + 1);
            inner[j] = inner_x && ly >= 0 && ly < wy;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int sx = SUB[b][0], sy = SUB[b][1];
                box[j][b] = lx >= -sx && lx <= wx - sx && ly >= -sy && ly <= wy - sy;
            }
        }
#pragma nounroll
        for (int lz = -1; lz <= wz; ++lz) {
            const int64_t plane = (int64_t)wrap_add(gz0 + lz, Lz) * plane_bytes;
            const bool inner_z = lz >= 0 && lz < wz;   // wave-uniform
            const uint8_t* at = lat + (lz + 1) * kPP;
            uint32_t c[4][4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    c[j][b] = at[src[j] + b * kArr + SUB[b][2] * kPP + SUB[b][1] * kP + SUB[b][0]];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint8_t* q = row[j] + plane;
                if (inner_z && inner[j])
                    gstore<uint32_t>(q, decode(c[j][0]) | decode(c[j][1]) << 8 | decode(c[j][2]) << 16 |
                                            decode(c[j][3]) << 24);
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const bool box_z = SUB[b][2] ? lz < wz : lz >= 0;
                    if (box_z && box[j][b] && !(inner_z && inner[j])) gstore<uint8_t>(q + b, (uint8_t)decode(c[j][b]));
                }
            }
        }
    }

    uint64_t sum = (uint64_t)dEsum;
    const uint32_t cnt = sums.nacc;   // already the wave's total
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)sum, o, kWave);
        const uint32_t hi = __shfl_xor((uint32_t)(sum >> 32), o, kWave);
        sum += (uint64_t)lo | ((uint64_t)hi << 32);
    }
    if (lane == 0) {
        unsigned long long* slot = (unsigned long long*)(D.state + (f % kSpread) * kSlotWords);
        if (sum) atomicAdd(slot, (unsigned long long)sum);
        if (cnt) atomicAdd(slot + 1, (unsigned long long)cnt);
    }
}

template <int WPG>
static hipError_t launch_fcc(const DevLattice* d_lat, const WorkItem* d_items, int n_groups, int t, int colour,
                             int smax, hipStream_t stream)
{
    const dim3 grid(xcd_grid(n_groups)), block(kWave * WPG);
    switch (smax) {
    case 1: hipLaunchKernelGGL((sweep_phase_fcc_kernel<1, WPG>), grid, block, 0, stream, d_lat, d_items, n_groups, t,
                               colour); break;
    case 2: hipLaunchKernelGGL((sweep_phase_fcc_kernel<2, WPG>), grid, block, 0, stream, d_lat, d_items, n_groups, t,
                               colour); break;
    case 3: hipLaunchKernelGGL((sweep_phase_fcc_kernel<3, WPG>), grid, block, 0, stream, d_lat, d_items, n_groups, t,
                               colour); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_sweep_phase_fcc(const DevLattice* d_lat, const WorkItem* d_items, int n_groups, int t, int colour,
                                  int smax, hipStream_t stream, int wpg)
{
    if (n_groups <= 0) return hipSuccess;
    if (wpg == kWavesPerGroupFccWide) {
        if (d_items) return hipErrorInvalidValue;   // work items cover kWavesPerGroupFcc blocks each
        return launch_fcc<kWavesPerGroupFccWide>(d_lat, d_items, n_groups, t, colour, smax, stream);
    }
    if (wpg != kWavesPerGroupFcc) return hipErrorInvalidValue;
    return launch_fcc<kWavesPerGroupFcc>(d_lat, d_items, n_groups, t, colour, smax, stream);
}

}  // namespace smcx
