// kernels.hip -- gfx950 kernels of libsmcx.
//
// sweep_phase: one colour phase of a Metropolis swap sweep (paper: Section
//   "Monte Carlo simulation", Eq. (3); link cells of Section "Distributed
//   SMC-X").  One wavefront owns one block of the shifted block grid: it
//   stages the block and its interaction halo from HBM into LDS, runs the 54
//   sub-colour rounds (64 lanes = the 4 x 4 x 4 same-residue cells of a 12-wide
//   block, one trial each), writes the block and the first-neighbour ring
//   back, and reduces its accepted energy changes.  Lanes of one round never
//   touch each other's sites, and LDS operations of one wavefront complete in
//   program order, so no barrier separates the rounds.
#include <type_traits>

#include "bcc_block.h"

namespace smcx {

// Waves per SIMD the BCC sweep kernel is compiled for (registers); LDS
// (4 block images and the weight planes per workgroup, 28.7 to 32.5 KB)
// admits 5 workgroups of 4 waves per CU, at K = 7, 8 and S = 3 (34 KB) 4.
constexpr int kSweepWavesPerSimd = 5;

// Offsets of the first shell from a corner site (body sites at cell offsets
// {-1,0}^3) and from a body site (corner sites at {0,+1}^3):
constexpr int kS1Corner = kArr;                      // + ex + ey*kP + ez*kPP, e in {0,1}
constexpr int kS1Body = -kArr - (kPP + kP + 1);      // + ex + ey*kP + ez*kPP, e in {0,1}

template <int SUB> __device__ __forceinline__ constexpr int s1base() { return SUB == 0 ? kS1Corner : kS1Body; }

// Shell offsets inside one sublattice array.
__device__ __forceinline__ constexpr int s2off(int k)
{
    return k == 0 ? 1 : k == 1 ? -1 : k == 2 ? kP : k == 3 ? -kP : k == 4 ? kPP : -kPP;
}
__device__ __forceinline__ constexpr int s3off(int k)
{
    // (+-1, +-1, 0), (+-1, 0, +-1), (0, +-1, +-1)
    return k == 0 ? 1 + kP : k == 1 ? 1 - kP : k == 2 ? -1 + kP : k == 3 ? -1 - kP
         : k == 4 ? 1 + kPP : k == 5 ? 1 - kPP : k == 6 ? -1 + kPP : k == 7 ? -1 - kPP
         : k == 8 ? kP + kPP : k == 9 ? kP - kPP : k == 10 ? -kP + kPP : -kP - kPP;
}

// First-shell offset (from the site) of neighbour e = ex + 2 ey + 4 ez.
template <int SUB> __device__ __forceinline__ constexpr int s1off(int e)
{
    return s1base<SUB>() + (e & 1) + ((e >> 1) & 1) * kP + ((e >> 2) & 1) * kPP;
}

// acc + sum over shells s < SMAX and fields p < NF of field(s, p) * w[s*KMAX + p],
// modulo 2^32: field = bias + n_i - n_j read from the packed difference
// (F = 5), or n_i - n_j from the two 4-bit fields (F = 4).  The constant may
// leave the int32 range for extreme tables while the true dE (|dE| < 2^29)
// never does: the 32-bit multiply-adds wrap, and the wrapped sum is exact.
template <int KMAX, int SMAX, int NF>
__device__ __forceinline__ uint32_t weigh(const uint32_t (&hi)[kMaxS], const uint32_t (&hj)[kMaxS],
                                          const int32_t* w, uint32_t acc)
{
    constexpr int PS = kPlane;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        if constexpr (Field<KMAX>::F == 5) {
            const uint32_t d = hi[s] - hj[s];   // fields 16 + n_i - n_j, no borrows
#pragma unroll
            for (int p = 0; p < NF; ++p)
                acc = mad24((d >> (5 * p)) & 31u, w[(s * KMAX + p) * PS], acc);
        } else {
#pragma unroll
            for (int p = 0; p < NF; ++p)
                acc = mad24((uint32_t)((int32_t)((hi[s] >> (4 * p)) & 15u) - (int32_t)((hj[s] >> (4 * p)) & 15u)),
                            w[(s * KMAX + p) * PS], acc);
        }
    }
    return acc;
}

// The codes of the cells around a lane's trials that the lane carries from
// one trial to the next along an x row of residue classes: corner(x), body(x),
// corner(x + 1), .. (three-shell trials).  Around the corner site (x, y, z):
//   a[e]   body(x - 1 + ex, y - 1 + ey, z - 1 + ez): the corner's first shell
//   c[e]   corner(x - 1 + ex, y + ey, z + ez) before the corner trial (its
//          own code is c[1]); corner(x + ex, ..), the body's first shell, after
//   xc     corner(x - 1, y - 1, z), (x, y - 1, z), (x - 1, y, z - 1),
//          (x, y, z - 1) before the corner trial; one cell on in x after it
//   xb     body(x - 1, y + 1, z), (x, y + 1, z), (x - 1, y, z + 1),
//          (x, y, z + 1) before the body trial; one cell on in x after it
// A trial finds its site, its partner, its first shell and 10 of its 18
// second and third neighbours here, and loads the cells that enter the window.
// Each trial puts its own changes into the window.  No other lane changes a
// cell while the window holds it: in units of a/2, the lanes' sites of a round
// are 6 apart on some axis, move along the row together, and a trial changes
// cells within 1 of its site, so only cells 5 or more from a lane's site are
// ever changed by another; every cell is within 2 of a site that reads it, and
// is taken in at most two trials (1 each along x) before and dropped at most
// two after.
//   pc, pb the packed counts (with the fields' bias) of the four cells of a
//          plane around the row's axis -- (x, y +- 1, z), (x, y, z +- 1) --
//          for the planes x - 1 and x of the corner (body) sublattice: four
//          third neighbours of the site one plane on, four second neighbours
//          of the plane's own site and four third neighbours of the next.
struct Window {
    uint32_t a[8], c[8], xb[4], xc[4], pc[2], pb[2];
    // The window before the corner trial at p = corner(x, y, z).
    __device__ __forceinline__ void load(const uint8_t* p, uint32_t bias)
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a[e] = p[kS1Corner + (e & 1) + (e >> 1 & 1) * kP + (e >> 2) * kPP];
            c[e] = e == 6 ? 0u : p[(e & 1) - 1 + (e >> 1 & 1) * kP + (e >> 2) * kPP];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            xc[k] = p[k - 1 - kP];
            xc[k + 2] = p[k - 1 - kPP];
            xb[k] = p[WavePitch::kBodyFromCorner + k - 1 + kP];
            xb[k + 2] = p[WavePitch::kBodyFromCorner + k - 1 + kPP];
        }
        // (hides from the compiler that the entries come from byte loads: it
        // would carry bytes and extend each again in every trial)
#pragma unroll
        for (int k = 0; k < 8; ++k) asm("" : "+v"(a[k]), "+v"(c[k]));
#pragma unroll
        for (int k = 0; k < 4; ++k) asm("" : "+v"(xb[k]), "+v"(xc[k]));
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            pc[k] = count4_from(bias, c[2 + k], xc[k], c[4 + k], xc[2 + k]);
            pb[k] = count4_from(bias, xb[k], a[4 + k], xb[2 + k], a[2 + k]);
        }
    }
};

// The code of the cell (I, J, K) from the site's cell in the other
// sublattice: from the window where it holds the cell, else loaded.
template <int SUB, int I, int J, int K>
__device__ __forceinline__ uint32_t other_cell(const uint8_t* lat, int ai, const Window& w)
{
    constexpr int kCell = (SUB == 0 ? 1 : -1) * WavePitch::kBodyFromCorner + I + J * kP + K * kPP;
    if constexpr (SUB == 0 && (I == -1 || I == 0) && J == 1 && K == 0) return w.xb[I + 1];
    else if constexpr (SUB == 0 && (I == -1 || I == 0) && J == 0 && K == 1) return w.xb[I + 3];
    else if constexpr (SUB == 1 && (I == 0 || I == 1) && J == -1 && K == 0) return w.xc[I];
    else if constexpr (SUB == 1 && (I == 0 || I == 1) && J == 0 && K == -1) return w.xc[I + 2];
    else return lat[ai + kCell];
}

// The cells of the site's own sublattice that a three-shell trial loads,
// whatever its direction: second and third neighbours (indices as s2off,
// s3off) and the cell that completes the next trial's first shell.
struct OwnCells {
    uint32_t r2_0, r3_0, r3_1, r3_4, r3_5, r3_8or11, r3_9, r3_10, fresh;
};
template <int SUB> __device__ __forceinline__ OwnCells load_own(const uint8_t* p)
{
    OwnCells o;
    o.r2_0 = p[s2off(0)];
    o.r3_0 = p[s3off(0)];
    o.r3_1 = p[s3off(1)];
    o.r3_4 = p[s3off(4)];
    o.r3_5 = p[s3off(5)];
    o.r3_9 = p[s3off(9)];
    o.r3_10 = p[s3off(10)];
    o.r3_8or11 = p[s3off(SUB == 0 ? 11 : 8)];
    o.fresh = p[SUB == 0 ? 1 + kP + kPP : 1 - kP - kPP];
    return o;
}

// Weigh the histograms (difference form: hi holds bias + n_i - n_j, hj is 0)
// with the pair's row and decide: returns the accepted lanes.  row: the
// byte-dot words, loaded ahead; w: the row in LDS for the other forms.
template <int KMAX, int SMAX, int MODE>
__device__ __forceinline__ int32_t energy_change(const uint32_t (&hi)[kMaxS], const uint32_t (&hj)[kMaxS],
                                                 const int32_t (&row)[3 * kMaxS + 1], const int32_t* w)
{
    if constexpr (MODE == kWtabDot) {
        // bytes 32 + n_i - n_j (bit 31, the last species, masked off) dotted
        // with the three base-256 digits of the folded weights, in one
        // chain: ((A2 * 256 + A1) * 256 + constant) + A0
        int32_t d[kMaxS];
#pragma unroll
        for (int s = 0; s < SMAX; ++s) d[s] = (int32_t)(KMAX == 5 ? hi[s] & 0x7fffffffu : hi[s]);   // (K <= 4: byte 3 weighs nothing)
        int32_t X = 0;
#pragma unroll
        for (int s = 0; s < SMAX; ++s) X = __builtin_amdgcn_sdot4(d[s], row[3 * s + 2], X, false);
        X = (int32_t)((uint32_t)X << 8);
#pragma unroll
        for (int s = 0; s < SMAX; ++s) X = __builtin_amdgcn_sdot4(d[s], row[3 * s + 1], X, false);
        X = (int32_t)(((uint32_t)X << 8) + (uint32_t)row[3 * SMAX]);
#pragma unroll
        for (int s = 0; s < SMAX; ++s) X = __builtin_amdgcn_sdot4(d[s], row[3 * s], X, false);
        return X;
    } else {
        // With kWtabDrop the rows fold in the last species, whose count
        // differences follow from the others (both sites have the same
        // number of neighbours per shell): only fields 0 .. KMAX-2 are read.
        return (int32_t)weigh<KMAX, SMAX, MODE == kWtabDrop ? KMAX - 1 : KMAX>(hi, hj, w,
                                                                               (uint32_t)w[SMAX * KMAX * kPlane]);
    }
}

// Row (a, b) of the weight planes, a = ci >> 5 and b = cj >> 5, at byte
// 4 (a*KMAX + b) of a plane.  (Lanes without a site in this round may decode
// stale halo bytes: their row still lies inside the planes, and their result
// is discarded.)
template <int KMAX>
__device__ __forceinline__ const int32_t* weight_row(const int32_t* wtab, uint32_t ci, uint32_t cj)
{
    const uint32_t row4 = __umul24(ci >> 5, 4u * KMAX) + ((cj >> 5) << 2);
    return (const int32_t*)((const uint8_t*)wtab + row4);
}

template <int KMAX, bool DOT>
constexpr uint32_t kFieldBias = DOT ? 0x20202020u
                              : Field<KMAX>::F == 5 ? 0x10u * (1u | 1u << 5 | 1u << 10 | 1u << 15 | 1u << 20 | 1u << 25) : 0u;

// What a three-shell trial leaves for after its direction's code.
struct TrialResult {
    int32_t dE;            // accepted change
    uint64_t swapped;      // lanes that changed the configuration
    uint32_t ci_new, next_plane;
    // (defined, with no instruction, where no direction has run yet)
    __device__ __forceinline__ TrialResult()
    {
        asm("" : "=v"(dE), "=s"(swapped), "=v"(ci_new), "=v"(next_plane));
    }
};

// One three-shell trial: the site at LDS byte ai (sublattice SUB), its partner
// first-shell neighbour E = ex + 2 ey + 4 ez (the direction shared by the
// round: the trial switches on it, wave-uniform, before anything else, so that
// each case is one straight line whose loads issue together).
//
// Half of the partner's neighbourhood is cells the site's own counts already
// hold.  In half-cell units j = i + s, s_a = +-1 the signs of E.  j's first
// shell is i + (0 or 2 s_a per axis): i, the site's second neighbours i + 2 s_a
// along the three axes, its third neighbours in the three planes with the same
// signs, and the far cell i + 2 s.  j's second and third shells hold the
// site's first-shell cells k with one or two direction bits flipped
// (popcount(k ^ E) = 1 or 2), counted once for both, and 3 and 9 cells beyond.
template <int KMAX, int SUB, int MODE, int E>
__device__ __forceinline__ void trial3(uint8_t* lat, int ai, const OwnCells& o, uint32_t u, uint64_t valid,
                                       const int32_t* wtab, const double* tab, float ln2kT, TrialResult& r, Window& w)
{
    constexpr bool DOT = MODE == kWtabDot;
    // 5-bit fields (and the byte-dot form) hold bias + n_i - n_j without
    // borrows: one packed difference per shell.  4-bit fields (KMAX = 8)
    // count the two neighbourhoods apart.
    constexpr bool DIFF = DOT || Field<KMAX>::F == 5;
    constexpr int ex = E & 1, ey = (E >> 1) & 1, ez = (E >> 2) & 1;
    constexpr int dx = ex ? 1 : -1, dy = ey ? 1 : -1, dz = ez ? 1 : -1;
    uint32_t (&s1)[8] = SUB == 0 ? w.a : w.c;
    const uint32_t ci = SUB == 0 ? w.c[1] : w.a[7], cj = s1[E];

    // ---- the rest of the trial's loads (o: those of every direction), then
    // every count ----
    uint32_t r2[6], r3[12];
    r2[0] = o.r2_0;
    r3[0] = o.r3_0;
    r3[1] = o.r3_1;
    r3[4] = o.r3_4;
    r3[5] = o.r3_5;
    r3[9] = o.r3_9;
    r3[10] = o.r3_10;
    if constexpr (SUB == 0) {
        r3[11] = o.r3_8or11;
        r2[1] = w.c[0]; r2[2] = w.c[3]; r2[3] = w.xc[1]; r2[4] = w.c[5]; r2[5] = w.xc[3];
        r3[2] = w.c[2]; r3[3] = w.xc[0]; r3[6] = w.c[4]; r3[7] = w.xc[2]; r3[8] = w.c[7];
    } else {
        r3[8] = o.r3_8or11;
        r2[1] = w.a[6]; r2[2] = w.xb[1]; r2[3] = w.a[5]; r2[4] = w.xb[3]; r2[5] = w.a[3];
        r3[2] = w.xb[0]; r3[3] = w.a[4]; r3[6] = w.xb[2]; r3[7] = w.a[2]; r3[11] = w.a[1];
    }
    // the partner's cells beyond the site's: the far one, 3 second and 9 third neighbours
    uint32_t q0, q2[3], q3[9];
    if constexpr (E == (SUB == 0 ? 7 : 1)) q0 = o.fresh;
    else q0 = lat[ai + dx + dy * kP + dz * kPP];
    constexpr int jx = SUB == 0 ? ex - 1 : ex, jy = SUB == 0 ? ey - 1 : ey, jz = SUB == 0 ? ez - 1 : ez;
    q2[0] = other_cell<SUB, jx + dx, jy, jz>(lat, ai, w);
    q2[1] = other_cell<SUB, jx, jy + dy, jz>(lat, ai, w);
    q2[2] = other_cell<SUB, jx, jy, jz + dz>(lat, ai, w);
    q3[0] = other_cell<SUB, jx + dx, jy + dy, jz>(lat, ai, w);
    q3[1] = other_cell<SUB, jx + dx, jy - dy, jz>(lat, ai, w);
    q3[2] = other_cell<SUB, jx - dx, jy + dy, jz>(lat, ai, w);
    q3[3] = other_cell<SUB, jx + dx, jy, jz + dz>(lat, ai, w);
    q3[4] = other_cell<SUB, jx + dx, jy, jz - dz>(lat, ai, w);
    q3[5] = other_cell<SUB, jx - dx, jy, jz + dz>(lat, ai, w);
    q3[6] = other_cell<SUB, jx, jy + dy, jz + dz>(lat, ai, w);
    q3[7] = other_cell<SUB, jx, jy + dy, jz - dz>(lat, ai, w);
    q3[8] = other_cell<SUB, jx, jy - dy, jz + dz>(lat, ai, w);
    const int32_t* wp = weight_row<KMAX>(wtab, ci, cj);
    int32_t row[3 * kMaxS + 1];
    if constexpr (DOT) {
#pragma unroll
        for (int k = 0; k < 3 * kMaxS + 1; ++k) row[k] = wp[k * kPlane];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- counts ----
    // Species histograms of both neighbourhoods (the partner is counted in
    // the first shell of i and i in that of j; the constant term undoes it).
    const Edges edges = edges_of(u, ln2kT);   // depends on the draw only
    // Cells of the window first, then the loaded ones in load order.
    constexpr uint32_t bias = kFieldBias<KMAX, DOT>;
    uint32_t hi[kMaxS], hj[kMaxS] = {0u, 0u, 0u};
    // the site's first shell but the partner and the cell opposite to it, by
    // the parity of the flipped direction bits: j's third- and second-shell
    // cells among them
    const uint32_t t_same = count3_from0(s1[E ^ 3], s1[E ^ 5], s1[E ^ 6]);
    const uint32_t t_other = count3_from0(s1[E ^ 1], s1[E ^ 2], s1[E ^ 4]);
    hi[0] = t_same + t_other + bias;
    count2<false>(hi[0], cj, s1[E ^ 7]);
    // second and third shell: the plane sums of the window, the next plane's,
    // and the cells at dx = 0 of the third shell
    uint32_t (&mine)[2] = SUB == 0 ? w.pc : w.pb;
    uint32_t (&others)[2] = SUB == 0 ? w.pb : w.pc;
    const uint32_t next_plane = count4_from(bias, r3[0], r3[1], r3[4], r3[5]);
    hi[2] = count4_from(0u - bias, r3[8], r3[9], r3[10], r3[11]);
    hi[2] += mine[0] + next_plane;
    hi[1] = count2_onto(mine[1], r2[1], r2[0]);
    uint32_t (&h)[kMaxS] = DIFF ? hi : hj;   // j's counts: subtracted from i's in the difference form
    count4<DIFF>(h[0], ci, r2[ex ? 0 : 1], r2[ey ? 2 : 3], r2[ez ? 4 : 5]);
    count4<DIFF>(h[0], r3[(ex ? 0 : 2) + (ey ? 0 : 1)], r3[4 + (ex ? 0 : 2) + (ez ? 0 : 1)],
                 r3[8 + (ey ? 0 : 2) + (ez ? 0 : 1)], q0);
    h[1] = DIFF ? h[1] - t_other : h[1] + t_other;
    h[2] = DIFF ? h[2] - t_same : h[2] + t_same;
    count3<DIFF>(h[1], q2[0], q2[1], q2[2]);
    count3<DIFF>(h[2], q3[0], q3[1], q3[2]);
    count3<DIFF>(h[2], q3[3], q3[4], q3[5]);
    count3<DIFF>(h[2], q3[6], q3[7], q3[8]);

    const int32_t dE = energy_change<KMAX, 3, MODE>(hi, hj, row, wp);
    const uint64_t acc = accepted_lanes(dE, u, edges, valid, tab);
    // Both bytes are stored by every lane (unchanged unless accepted): no two
    // lanes of a round touch the same byte.
    const bool accept = __builtin_amdgcn_inverse_ballot_w64(acc);
    const uint32_t ci_new = accept ? cj : ci, cj_new = accept ? ci : cj;
    lat[ai] = (uint8_t)ci_new;
    lat[ai + s1off<SUB>(E)] = (uint8_t)cj_new;
    r.dE = accept ? dE : 0;   // (0 for equal species: their row is zero)
    r.swapped = __builtin_amdgcn_ballot_w64(ci != cj) & acc;
    r.ci_new = ci_new;
    r.next_plane = next_plane;
    s1[E] = cj_new;
    if constexpr (E == 2 || E == 3 || E == 4 || E == 5)   // the partner is a cell of a plane sum
        others[E & 1] = count_swap(others[E & 1], cj_new, cj);
}

// The window of the next trial, and the trial's changes summed: the same for
// every direction.
template <int SUB>
__device__ __forceinline__ void advance(Window& w, const OwnCells& o, const TrialResult& r, Sums& sums)
{
    sums.dE += r.dE;
    sums.nacc += (uint32_t)__popcll(r.swapped);
    const Window v = w;
    if constexpr (SUB == 0) {
        w.pc[0] = v.pc[1];
        w.pc[1] = r.next_plane;
        w.c[0] = r.ci_new;
        w.c[1] = o.r2_0;
        w.c[2] = v.c[3];
        w.c[3] = o.r3_0;
        w.c[4] = v.c[5];
        w.c[5] = o.r3_4;
        w.c[6] = v.c[7];
        w.c[7] = o.fresh;
        w.xc[0] = v.xc[1];
        w.xc[1] = o.r3_1;
        w.xc[2] = v.xc[3];
        w.xc[3] = o.r3_5;
    } else {
        w.pb[0] = v.pb[1];
        w.pb[1] = r.next_plane;
        w.a[0] = v.a[1];
        w.a[1] = o.fresh;
        w.a[2] = v.a[3];
        w.a[3] = o.r3_5;
        w.a[4] = v.a[5];
        w.a[5] = o.r3_1;
        w.a[6] = r.ci_new;
        w.a[7] = o.r2_0;
        w.xb[0] = v.xb[1];
        w.xb[1] = o.r3_0;
        w.xb[2] = v.xb[3];
        w.xb[3] = o.r3_4;
    }
}

// One trial with one or two shells, direction e (wave-uniform): the partner
// and both neighbourhoods are loaded.
template <int KMAX, int SMAX, int SUB, int MODE>
__device__ __forceinline__ void trial12(uint8_t* lat, int ai, uint32_t u, int e, uint64_t valid, const int32_t* wtab,
                                        const double* tab, float ln2kT, Sums& sums)
{
    constexpr bool DOT = MODE == kWtabDot;
    constexpr bool DIFF = DOT || Field<KMAX>::F == 5;
    const int aj = ai + s1base<SUB>() + (e & 1) + ((e >> 1) & 1) * kP + ((e >> 2) & 1) * kPP;
    const uint32_t ci = lat[ai], cj = lat[aj];
    uint32_t n1[8], n2[6], p1[8], p2[6];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        n1[k] = lat[ai + s1off<SUB>(k)];
        p1[k] = lat[aj + s1off<1 - SUB>(k)];
    }
    if constexpr (SMAX == 2) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            n2[k] = lat[ai + s2off(k)];
            p2[k] = lat[aj + s2off(k)];
        }
    }
    const int32_t* wp = weight_row<KMAX>(wtab, ci, cj);
    int32_t row[3 * kMaxS + 1];
    if constexpr (DOT) {
#pragma unroll
        for (int k = 0; k < 3 * SMAX + 1; ++k) row[k] = wp[k * kPlane];
    }
    __builtin_amdgcn_sched_barrier(0);
    const Edges edges = edges_of(u, ln2kT);
    constexpr uint32_t bias = kFieldBias<KMAX, DOT>;
    uint32_t hi[kMaxS], hj[kMaxS] = {0u, 0u, 0u};
    uint32_t (&h)[kMaxS] = DIFF ? hi : hj;
    hi[0] = count4_from(bias, n1[0], n1[1], n1[2], n1[3]);
    count4<false>(hi[0], n1[4], n1[5], n1[6], n1[7]);
    count4<DIFF>(h[0], p1[0], p1[1], p1[2], p1[3]);
    count4<DIFF>(h[0], p1[4], p1[5], p1[6], p1[7]);
    if constexpr (SMAX == 2) {
        hi[1] = count4_from(bias, n2[0], n2[1], n2[2], n2[3]);
        count2<false>(hi[1], n2[4], n2[5]);
        count3<DIFF>(h[1], p2[0], p2[1], p2[2]);
        count3<DIFF>(h[1], p2[3], p2[4], p2[5]);
    }
    const int32_t dE = energy_change<KMAX, SMAX, MODE>(hi, hj, row, wp);
    const uint64_t acc = accepted_lanes(dE, u, edges, valid, tab);
    const bool accept = __builtin_amdgcn_inverse_ballot_w64(acc);
    lat[ai] = (uint8_t)(accept ? cj : ci);
    lat[aj] = (uint8_t)(accept ? ci : cj);
    sums.dE += accept ? dE : 0;
    sums.nacc += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(ci != cj) & acc);
}

// One trial with the round's direction e (wave-uniform).  Tests of e's top
// bit, then of the four directions, one after the other, each a compare and a
// branch over the code it guards: as a switch the compiler makes every level
// of the tree a chain of flags and branches.  The empty asm keeps it from
// threading the tests together again.  What every direction leaves goes
// through TrialResult, so that the joins merge few registers: with the whole
// window updated inside the arms the tests lost 1.2 % to the switch, this way
// they gain (512^3: 4.27 to 4.23 ms for 4 sweeps; 512 x 512 x 64 slab: 1.77 to
// 1.75 for 5).
template <int KMAX, int SUB, int MODE, int E0>
__device__ __forceinline__ void trial3_of_four(int e, uint8_t* lat, int ai, const OwnCells& o, uint32_t u,
                                               uint64_t valid, const int32_t* wtab, const double* tab, float ln2kT,
                                               TrialResult& r, Window& w)
{
    if (e == E0) trial3<KMAX, SUB, MODE, E0>(lat, ai, o, u, valid, wtab, tab, ln2kT, r, w);
    asm volatile("" : "+s"(e));
    if (e == E0 + 1) trial3<KMAX, SUB, MODE, E0 + 1>(lat, ai, o, u, valid, wtab, tab, ln2kT, r, w);
    asm volatile("" : "+s"(e));
    if (e == E0 + 2) trial3<KMAX, SUB, MODE, E0 + 2>(lat, ai, o, u, valid, wtab, tab, ln2kT, r, w);
    asm volatile("" : "+s"(e));
    if (e == E0 + 3) trial3<KMAX, SUB, MODE, E0 + 3>(lat, ai, o, u, valid, wtab, tab, ln2kT, r, w);
}
template <int KMAX, int SMAX, int SUB, int MODE>
__device__ __forceinline__ void trial(uint8_t* lat, int ai, uint32_t u, int e, uint64_t valid, const int32_t* wtab,
                                      const double* tab, float ln2kT, Sums& sums, Window& w)
{
    if constexpr (SMAX == 3) {
        const OwnCells o = load_own<SUB>(lat + ai);
        TrialResult r;
        if (e < 4) trial3_of_four<KMAX, SUB, MODE, 0>(e, lat, ai, o, u, valid, wtab, tab, ln2kT, r, w);
        asm volatile("" : "+s"(e));
        if (e >= 4) trial3_of_four<KMAX, SUB, MODE, 4>(e, lat, ai, o, u, valid, wtab, tab, ln2kT, r, w);
        advance<SUB>(w, o, r, sums);
    } else {
        trial12<KMAX, SMAX, SUB, MODE>(lat, ai, u, e, valid, wtab, tab, ln2kT, sums);
    }
}

// ---------------------------------------------------------------------------
// What bounds it (512^3, K = 5, S = 3, a colour launch of N/8 trials): issue of
// vector and LDS instructions together.  The launch took 164 us when each
// trial loaded 32 cells; with the row window (fewer loads, plane sums in place
// of single counts), scalar decision masks and the set-up reads overlapped it
// takes 134 us (mean of 200 sweeps at 800 K; 138 in the first 20): 108 VALU,
// 36 LDS and 44 scalar instructions per wave-round, no bank conflicts.  Staging, set-up and write-back are about a third of a
// wave's time in the first generation of a launch.
// SLAB: the lattice is a z-slab (DevLattice::slab) -- its own instance, so
// the periodic kernel carries none of the slab's addressing.  A workgroup
// takes kWavesPerGroup blocks, one wave each.  Wider workgroups (3 of 7 or 2
// of 11 per CU, 21 and 22 waves) fill the wave slots of a 512^3 colour launch
// more evenly but measured no faster: a CU is busy issuing at 20 waves.
template <int KMAX, int SMAX, bool SLAB>
__global__ __launch_bounds__(kWave * kWavesPerGroup) __attribute__((amdgpu_waves_per_eu(kSweepWavesPerSimd)))
void sweep_phase_kernel(const DevLattice* __restrict__ lats, const WorkItem* __restrict__ items, int n_groups,
                        int t, int colour)
{
    // One LDS buffer: the weight planes at offset 0 (so a plane's LDS offset
    // fits the st64 immediates of ds_read2st64_b32 and row addresses need no
    // base added), then the block images.
    constexpr int kWBytes = wplanes(KMAX, SMAX) * kPlane * 4;
    __shared__ __attribute__((aligned(16))) uint8_t s_mem[kWBytes + kWavesPerGroup * kWaveLds];
    int32_t* s_w = (int32_t*)s_mem;
    uint8_t* s_lat = s_mem + kWBytes;

    const int wave = wave_id();
    const int lane = threadIdx.x % kWave;
    // group grp of the launch's n_groups (XCD-aware order): a work item of a
    // batched launch, or kWavesPerGroup blocks in a row of a single lattice
    const int grp = xcd_group(n_groups);
    if (grp < 0) return;   // no later barrier in a workgroup without a group
    int li = 0, f = grp * kWavesPerGroup;
    if (items) {
        li = items[grp].lattice;
        f = items[grp].first_block;
    }
    const DevLattice& D = lats[li];
    const uint32_t s = D.sweep0 + (uint32_t)t;

    // The words of the weight planes, on their way while the block is set up.
    // The threshold tables of sweep s stay in global memory (read only for the
    // few draws whose decision needs them), which leaves LDS for five
    // workgroups per CU.
    constexpr int kThreads = kWave * kWavesPerGroup;
    constexpr int kWords = wplanes(KMAX, SMAX) * kPlane, kWPer = (kWords + kThreads - 1) / kThreads;
    int32_t wword[kWPer];
#pragma unroll
    for (int n = 0; n < kWPer; ++n) {
        const int k = n * kThreads + (int)threadIdx.x, row = k % kPlane;
        wword[n] = k < kWords && row < KMAX * KMAX ? D.wtab[row * wrow(KMAX, SMAX) + k / kPlane] : 0;
    }
    int ti = (int)(s - D.tab_s0);
    ti = ti < 0 ? 0 : (ti >= D.n_tabs ? D.n_tabs - 1 : ti);
    const double* g_tab = D.tabs + (size_t)ti * kTab;

    f += wave;
    const bool active = f < D.blocks_per_colour;   // wave-uniform; the group's last waves may have no block
    const uint32_t k0 = D.key[0], k1 = D.key[1];
    const BccDraws pb = bcc_draws(s, colour, k0, k1, lane);
    const BccBlock B = bcc_block<SLAB>(D, active ? f : 0, colour, pb);
    uint8_t* lat = s_lat + wave * kWaveLds;
    const bool dot_codes = KMAX <= 5 && D.drop_last == kWtabDot;
    auto put_weights = [&] {
#pragma unroll
        for (int n = 0; n < kWPer; ++n) {
            const int k = n * kThreads + (int)threadIdx.x;
            if (k < kWords) s_w[k] = wword[n];
        }
    };
    if (active) bcc_stage<KMAX, WavePitch, SLAB, 1>(B, lat, lane, 0, dot_codes, put_weights);
    else put_weights();
    __syncthreads();
    if (!active) return;   // no later barrier

    // ---- 27 residue classes x 2 sublattices = 54 rounds ----
    // Lane (ix, iy, iz) takes local cell (rx + 3 ix, ry + 3 iy, rz + 3 iz) of
    // residue class m = (rz*3 + ry)*3 + rx; lanes past the block edge only
    // compute.  Acceptance draws: one Philox call per lane and residue pair
    // (2k, 2k+1), counter (base cell, s, colour + 256 k), the base cell being
    // the lane's cell of class 0; class 2k takes words 0 (corner) and 1
    // (body), class 2k+1 words 2 and 3.  The partner direction of sub-colour
    // q = 2m + b, the same for all blocks of the colour: x step bit q of the
    // Philox call (0, 0, s, 40 + colour), y and z steps bits 2q and 2q+1 of
    // the call (0, 0, s, 32 + colour).
    int ix, iy, iz;
    lane_cell(lane, ix, iy, iz);
    const int lane_c = (3 * iz + 1) * kPP + (3 * iy + 1) * kP + (3 * ix + 1);
    constexpr int kBodyFromCorner = kArr + kPP + kP + 1;
    uint32_t base_lo, base_hi;
    bcc_base_cell<SLAB>(B, D.z_off, ix, iy, iz, base_lo, base_hi);
    int64_t dEsum = 0;
    Sums sums = {0, 0u};
    const float ln2kT = (float)g_tab[kTabLn2kT];
    // The rounds, instantiated for each form of the weight rows (byte-dot or
    // full for KMAX <= 5, folded or full above): the form is per lattice, so
    // each instance stays branch-free.
    auto all_rounds = [&](auto mode_tag) {
        constexpr int MODE = decltype(mode_tag)::value;
        Window win;
        // A loop over the nine x rows of classes, each row's three classes
        // unrolled: the window's cells then change registers, not places (a
        // loop over classes moved 14 of them per trial).  The row's code, 6 x
        // 8 directions, is 36 KB of the 64 KB instruction cache that two CUs
        // share; all waves of a launch run the same directions.
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        int ac = lane_c, ry = 0, rz = 0;
#pragma nounroll
        for (int m0 = 0; m0 < 27; m0 += 3) {
            const uint64_t valid_yz = __builtin_amdgcn_ballot_w64((3 * iy < B.wy - ry) & (3 * iz < B.wz - rz));
            // partner directions: bits 2m, 2m + 1 of x, 4m .. 4m + 3 of yz
            uint32_t xb = (uint32_t)(pb.x >> (2 * m0));
            uint32_t b4 = (uint32_t)(m0 < 16 ? pb.yz_lo >> (4 * m0) : pb.yz_hi >> (4 * m0 - 64));
            if (m0 == 15) b4 |= (uint32_t)pb.yz_hi << 4;   // (class 15 ends the low word)
            if constexpr (SMAX == 3) win.load(lat + ac, kFieldBias<KMAX, MODE == kWtabDot>);
            auto one_class = [&](auto rx_tag) {
                constexpr int rx = decltype(rx_tag)::value;
                // one Philox call per pair of classes
                if (((m0 + rx) & 1) == 0) {
                    w[0] = base_lo; w[1] = base_hi; w[2] = s;
                    w[3] = (uint32_t)colour + 256u * (uint32_t)((m0 + rx) >> 1);
                    philox4x32_10(w, k0, k1);
                }
                const uint32_t u0 = w[0], u1 = w[1];
                w[0] = w[2];
                w[1] = w[3];
                const int e0 = (int)(xb & 1u) | (int)(b4 & 3u) << 1;
                const int e1 = (int)((xb >> 1) & 1u) | (int)((b4 >> 2) & 3u) << 1;
                xb >>= 2;
                b4 >>= 4;
                const uint64_t valid = valid_yz & __builtin_amdgcn_ballot_w64(3 * ix < B.wx - rx);
                trial<KMAX, SMAX, 0, MODE>(lat, ac + rx, u0, e0, valid, s_w, g_tab, ln2kT, sums, win);
                __builtin_amdgcn_wave_barrier();
                trial<KMAX, SMAX, 1, MODE>(lat, ac + rx + kBodyFromCorner, u1, e1, valid, s_w, g_tab, ln2kT, sums, win);
                __builtin_amdgcn_wave_barrier();
                dEsum += (int64_t)sums.dE;
                sums.dE = 0;
            };
            one_class(std::integral_constant<int, 0>{});
            one_class(std::integral_constant<int, 1>{});
            one_class(std::integral_constant<int, 2>{});
            ac += kP;
            if (++ry == 3) {
                ry = 0;
                ++rz;
                ac += kPP - 3 * kP;
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

    bcc_write_back<WavePitch, SLAB, 1>(B, lat, lane, 0);

    // ---- wavefront reduction of the energy change and accepted count ----
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

int kmax_for(int K)
{
    if (K <= 2) return 2;
    if (K <= 3) return 3;
    if (K <= 4) return 4;
    if (K <= 5) return 5;
    if (K <= 6) return 6;
    return 8;
}

template <int KMAX, int SMAX, bool SLAB>
static hipError_t launch_t(const DevLattice* d_lat, const WorkItem* d_items, int n_groups, int t,
                           int colour, hipStream_t stream)
{
    hipLaunchKernelGGL((sweep_phase_kernel<KMAX, SMAX, SLAB>), dim3(xcd_grid(n_groups)),
                       dim3(kWave * kWavesPerGroup), 0, stream, d_lat, d_items, n_groups, t, colour);
    return hipGetLastError();
}

template <int KMAX, bool SLAB>
static hipError_t launch_k(const DevLattice* d_lat, const WorkItem* d_items, int n_groups, int t,
                           int colour, int smax, hipStream_t stream)
{
    switch (smax) {
    case 1: return launch_t<KMAX, 1, SLAB>(d_lat, d_items, n_groups, t, colour, stream);
    case 2: return launch_t<KMAX, 2, SLAB>(d_lat, d_items, n_groups, t, colour, stream);
    case 3: return launch_t<KMAX, 3, SLAB>(d_lat, d_items, n_groups, t, colour, stream);
    }
    return hipErrorInvalidValue;
}

template <bool SLAB>
static hipError_t launch_bcc(const DevLattice* d_lat, const WorkItem* d_items, int n_groups, int t, int colour,
                             int kmax, int smax, hipStream_t stream)
{
    switch (kmax) {
    case 2: return launch_k<2, SLAB>(d_lat, d_items, n_groups, t, colour, smax, stream);
    case 3: return launch_k<3, SLAB>(d_lat, d_items, n_groups, t, colour, smax, stream);
    case 4: return launch_k<4, SLAB>(d_lat, d_items, n_groups, t, colour, smax, stream);
    case 5: return launch_k<5, SLAB>(d_lat, d_items, n_groups, t, colour, smax, stream);
    case 6: return launch_k<6, SLAB>(d_lat, d_items, n_groups, t, colour, smax, stream);
    case 8: return launch_k<8, SLAB>(d_lat, d_items, n_groups, t, colour, smax, stream);
    }
    return hipErrorInvalidValue;
}

// Colour launches of at most this many blocks give a block four waves
// (kernels_split.hip).  Their time rises by a step with every 256 blocks
// (another workgroup on each CU; LDS holds three, or four where the weight
// planes are few), while one wave per block takes nearly the same time up to
// 1,024 blocks (a workgroup of four blocks to each CU).  us per launch on 256
// CUs, one wave per block against four:
//   blocks         64           512          576          729          800
//   K = 5, S = 3   31.0  19.1   32.4  26.1   32.4  33.0   32.9  33.6   32.9  43.0
//   K = 8, S = 3   43.2  27.0   44.5  36.6   44.4  47.7   44.9  48.2   44.9  63.9
//   K = 8, S = 2   33.0  21.7   34.5  28.6   34.4  35.7   35.0  36.2   35.1  48.6
//   K = 5, S = 2   26.6  17.0   28.0  22.6   28.1  27.5   28.7  28.1   28.7  32.9
//   K = 2, S = 1   22.6  15.4   24.1  19.6   24.1  22.9   24.7  23.5   24.7  27.2
// The lines cross between 512 and 513 blocks for the heavier trials.  With two
// shells and K <= 5, or one shell, they cross between 768 and 769: the one
// line for all leaves 1 to 5 % there to the four waves.
constexpr int kSplitBlocks = 512;
// FCC (35 to 37 KB of LDS, four workgroups to a CU; kernels_fcc_split.hip), us
// per launch, one wave per block against four:
//   blocks         64           512          729          800          1,000        1,100
//   K = 5, S = 3   79.4  42.9   80.4  58.8   94.1  78.4   94.8  96.8   95.4  97.5   100.9 117.8
//   K = 3, S = 2   60.1  35.2   62.4  45.5   72.4  56.8   72.6  68.1   73.0  68.6   73.5  84.5
//   K = 3, S = 1   54.9  31.5   56.9  39.5   66.0  48.6   66.0  57.3   66.7  57.9   66.7  71.9
// At three shells the lines cross between 768 and 769 blocks, with fewer
// between 1,024 and 1,025: the one line for all leaves 6 (S = 2) to 15 % (S = 1)
// of such a launch to the four waves.
constexpr int kSplitBlocksFcc = 768;

hipError_t launch_sweep_phase(int lattice, const DevLattice* d_lat, const WorkItem* d_items, int n_groups, int n_blocks,
                              int t, int colour, int kmax, int smax, hipStream_t stream, bool slab, int wpg)
{
    if (n_groups <= 0) return hipSuccess;
    if (lattice == 1 && !slab && n_blocks <= kSplitBlocksFcc)
        return launch_sweep_split_fcc(d_lat, d_items, d_items ? n_groups * kWavesPerGroupFcc : n_blocks, t, colour, smax,
                                      stream);
    if (lattice == 1)
        return slab ? hipErrorInvalidValue
                    : launch_sweep_phase_fcc(d_lat, d_items, n_groups, t, colour, smax, stream,
                                             wpg ? wpg : kWavesPerGroupFcc);
    if (wpg && wpg != kWavesPerGroup) return hipErrorInvalidValue;
    if (n_blocks <= kSplitBlocks)
        return launch_sweep_split(d_lat, d_items, d_items ? n_groups * kWavesPerGroup : n_blocks, t, colour, kmax, smax,
                                  stream, slab);
    if (slab) return launch_bcc<true>(d_lat, d_items, n_groups, t, colour, kmax, smax, stream);
    return launch_bcc<false>(d_lat, d_items, n_groups, t, colour, kmax, smax, stream);
}

__global__ void species_max_kernel(const uint8_t* __restrict__ g, size_t n, unsigned int* __restrict__ out)
{
    unsigned int m = 0;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        m = max(m, (unsigned int)g[i]);
    for (int o = 32; o >= 1; o >>= 1) m = max(m, (unsigned int)__shfl_xor(m, o, kWave));
    if ((threadIdx.x % kWave) == 0) atomicMax(out, m);
}

hipError_t launch_species_max(const uint8_t* species, size_t n, unsigned int* d_max, hipStream_t stream)
{
    size_t groups = (n + 255) / 256;
    if (groups > 4096) groups = 4096;
    if (groups == 0) groups = 1;
    hipLaunchKernelGGL(species_max_kernel, dim3((unsigned)groups), dim3(256), 0, stream, species, n, d_max);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Verification hooks: the device's FP64 threshold products and Philox.
__global__ void thresholds_kernel(const double* __restrict__ tab, const int32_t* __restrict__ dE, int n,
                                  double* __restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int e = dE[k] < 1 ? 1 : (dE[k] > (1 << 24) - 1 ? (1 << 24) - 1 : dE[k]);
    out[k] = (tab[512 + (e >> 16)] * tab[256 + ((e >> 8) & 255)]) * tab[e & 255];
}

hipError_t launch_thresholds(const double* d_tab, const int32_t* d_dE, int n, double* d_out, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(thresholds_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, d_tab, d_dE, n, d_out);
    return hipGetLastError();
}

__global__ void accept_bounds_kernel(const double* __restrict__ tab, const uint32_t* __restrict__ u, int n,
                                     int32_t* __restrict__ lo, int32_t* __restrict__ hi)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int a, b;
    accept_bounds(u[k], (float)tab[kTabLn2kT], a, b);
    lo[k] = a;
    hi[k] = b;
}

hipError_t launch_accept_bounds(const double* d_tab, const uint32_t* d_u, int n, int32_t* d_lo, int32_t* d_hi,
                                hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(accept_bounds_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, d_tab, d_u, n, d_lo, d_hi);
    return hipGetLastError();
}

// Exhaustive check of the acceptance bounds over every 32-bit draw u (the
// acceptance draws of both lattices).  For each u the
// kernel forms the edges as the sweep kernels do; the largest dE they accept
// without the table is lo = floor(elo) and the smallest they reject without
// it is hi + 1, hi = floor(ehi).  It evaluates the exact test of Eq. (3) on
// the FP64 table products at dE = lo, lo - 1 (must accept) and hi + 1,
// hi + 2 (must reject), for those dE in (0, 2^24).
// out[0] counts draws violating the lower bound, out[1] the upper bound,
// out[2] holds the largest |(32 - log2 float(u)) - (32 - log2 u)| as the
// bits of a non-negative double (u > 0), out[3] the widest band hi - lo.
__global__ __launch_bounds__(256) void accept_bounds_check_kernel(const double* __restrict__ tab,
                                                                  unsigned long long* __restrict__ out)
{
    const float c = (float)tab[kTabLn2kT];
    unsigned long long bad_lo = 0, bad_hi = 0;
    double max_err = 0.0;
    int max_band = 0;
    auto thr = [&](int e) {
        return (tab[512 + (e >> 16)] * tab[256 + ((e >> 8) & 255)]) * tab[e & 255];
    };
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < (1ull << 32); v += stride) {
        const uint32_t u = (uint32_t)v;
        float elo, ehi;
        accept_edges(u, c, elo, ehi);
        const int lo = (int)fminf(floorf(elo), 1.0e9f), hi = (int)fminf(floorf(ehi), 1.0e9f);
        max_band = max(max_band, hi - lo);
        if (u == 0u) continue;   // the kernels always consult the table for u = 0
        const double du = (double)u;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int a = lo - k, b = hi + 1 + k;
            if (a > 0 && a < (1 << 24) && !(du < thr(a))) ++bad_lo;
            if (b > 0 && b < (1 << 24) && (du < thr(b))) ++bad_hi;
        }
        const double l = (double)(32.0f - __builtin_amdgcn_logf((float)u));
        max_err = fmax(max_err, fabs(l - (32.0 - log2(du))));
    }
    for (int o = 32; o >= 1; o >>= 1) {
        bad_lo += __shfl_xor(bad_lo, o, kWave);
        bad_hi += __shfl_xor(bad_hi, o, kWave);
        max_err = fmax(max_err, __shfl_xor(max_err, o, kWave));
        max_band = max(max_band, __shfl_xor(max_band, o, kWave));
    }
    if ((threadIdx.x % kWave) == 0) {
        if (bad_lo) atomicAdd(&out[0], bad_lo);
        if (bad_hi) atomicAdd(&out[1], bad_hi);
        atomicMax(&out[2], (unsigned long long)__double_as_longlong(max_err));
        atomicMax(&out[3], (unsigned long long)max_band);
    }
}

hipError_t launch_accept_bounds_check(const double* d_tab, unsigned long long* d_out, hipStream_t stream)
{
    hipLaunchKernelGGL(accept_bounds_check_kernel, dim3(8192), dim3(256), 0, stream, d_tab, d_out);
    return hipGetLastError();
}

__global__ void philox_kernel(const uint32_t* __restrict__ ctr, uint32_t k0, uint32_t k1, int n,
                              uint32_t* __restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    uint32_t c[4] = {ctr[4 * k], ctr[4 * k + 1], ctr[4 * k + 2], ctr[4 * k + 3]};
    philox4x32_10(c, k0, k1);
    for (int w = 0; w < 4; ++w) out[4 * k + w] = c[w];
}

hipError_t launch_philox(const uint32_t* d_ctr, uint32_t k0, uint32_t k1, int n, uint32_t* d_out,
                         hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(philox_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, d_ctr, k0, k1, n, d_out);
    return hipGetLastError();
}

}  // namespace smcx
