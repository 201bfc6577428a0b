// lbm_march.h -- T time steps of a strip of columns in one pass down its rows, in registers.
//
// One wave owns a strip of 64 columns (one column per lane) and a segment of rows, and walks the
// rows from below. Every row that it loads enters the first of T time levels; each level holds
// what it needs of the last rows in registers, and the populations that a level's collision
// produces stream straight into the next level's pull: to the same lane's registers, or to the
// neighbouring lane's through a cross-lane move. No level touches memory but the first (one read
// of every population) and the last (one write), and there is no LDS and no barrier, so the wave's
// T collision chains per row are bounded by arithmetic issue alone.
//
// Level t (0 .. T-1) of row p: with the 9 pulled populations f of row p, rho and psi are formed,
// then row c = p - 1 collides (its own f was held, psi of rows c-1, c, c+1 is known) and its f*
// completes the pull of row c - 1 = p - 2 at level t + 1. The halo is 2T-1 columns on each side
// and 2T-1 rows above and below (the outermost only pulled): lanes within 2t+1 of the strip's edge
// hold values of no meaning after level t, which no lane that is stored ever reads.
//
// What bounds it: T = 3 moves 48 bytes per update where the two-step tiles move 72, and a level
// issues 180 vector instructions per row (195 with two viscosities) against 350 per node and step of
// the tiles (each psi and each pull is made once; the halo costs 10 of 64 lanes). On 4096 x 4096
// (2.4 GB) a launch takes 640 us: the vector units are busy 70% of it and memory moves 2.7 GB
// (4.3 TB/s; a plain copy reaches 5.2), where two steps of tiles took 622 us. T = 2 is bound by memory
// alone (600 us per launch), T = 4 spills 70 registers (of 256 at two waves per SIMD) and runs 2.5
// times longer. The next row's loads are issued one row ahead into registers; a ring of three rows in
// LDS filled by direct loads (4 bytes a lane) freed 18 registers and was 3% slower.
//
// The arithmetic of every node is that of step_tile (sum9, psi_of_rho, cohesion_sum, collide), so
// the bits are those of T single steps.
#pragma once
#include <type_traits>

#include "lbm_device.h"

namespace lbm {

// Columns that a strip of T levels stores: the 64 lanes less 2T-1 on each side.
__host__ __device__ constexpr int march_cols(int T) { return 64 - 2 * (2 * T - 1); }

// Starts the loads of the pull of row y (a fluid row of the lattice) into f. b: byte offsets in a
// row of this lane's column and of its left and right neighbours. PLAIN: no neighbour of the row
// is a solid row or reached through the periodic seam.
template <bool PLAIN, class X>
__device__ __forceinline__ void march_load(const KParams& P, const double* __restrict__ g,
                                           const unsigned (&b)[3], int y, double f[9]) {
    const long long pl = P.plane;
    const bool bot = !PLAIN && P.walls && y == 1, top = !PLAIN && P.walls && y == P.ny - 2;
    int ym = y - 1, yp = y + 1;
    if (!PLAIN && !P.walls) {
        ym = y > 0 ? y - 1 : P.ny - 1;
        yp = y < P.ny - 1 ? y + 1 : 0;
    }
    const double* r0 = g + (long long)y * P.pitch;
    const double* rm = g + (long long)ym * P.pitch;
    const double* rp = g + (long long)yp * P.pitch;
    // opaque offsets: the address stays a scalar base plus a 32-bit lane offset
    unsigned o[3] = {b[0], b[1], b[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k) X::opaque(o[k]);
    auto at = [&](const double* r, int a, unsigned off) {
        return *(const double*)((const char*)(r + a * pl) + off);
    };
    f[0] = at(r0, 0, o[0]);
    f[1] = at(r0, 1, o[1]);
    f[3] = at(r0, 3, o[2]);
    if (bot) {  // reflected at the bottom wall
        f[2] = at(r0, 4, o[0]);
        f[5] = at(r0, 7, o[0]);
        f[6] = at(r0, 8, o[0]);
    } else {
        f[2] = at(rm, 2, o[0]);
        f[5] = at(rm, 5, o[1]);
        f[6] = at(rm, 6, o[2]);
    }
    if (top) {  // reflected at the top wall
        f[4] = at(r0, 2, o[0]);
        f[7] = at(r0, 5, o[0]);
        f[8] = at(r0, 6, o[0]);
    } else {
        f[4] = at(rp, 4, o[0]);
        f[7] = at(rp, 7, o[2]);
        f[8] = at(rp, 8, o[1]);
    }
}

// What a level keeps between rows.
struct MarchLevel {
    double f[9], rho;      // pulled populations and density of row p - 1
    double w0[3], w1[3];   // psi of rows p - 2 and p - 1 at the left, own and right column
    double up[3];          // next level's pull of row c: f2, f5, f6 (from row c - 1)
    double a[6];           // next level's pull of row c - 1: f2, f5, f6, f0, f1, f3
    double F[2];           // wet-node wall: the last boundary node's force
};

// T steps of the columns [x0, x0 + march_cols(T)) and rows [y0, y1] of one lattice, by the 64
// lanes of a wave (all active). lane: this lane's index; X: the wave's cross-lane
// moves (X::left(v) is v of the lane to the left). x0, y0, y1 are uniform. VISC as in
// collide_force.
template <int T, int GEO, int EOS, int VISC, class X>
__device__ __forceinline__ void march_strip(const KParams& P, const double* __restrict__ gin,
                                            double* __restrict__ gout,
                                            const double* __restrict__ gw, int x0, int y0, int y1,
                                            int lane) {
    static_assert(GEO != GEO_MASK, "rows of solid nodes only");
    constexpr int H = 2 * T - 1;
    const int x = x0 - H + lane;
    const unsigned xc = wrapx(x, P.nx);
    const bool store = lane >= H && lane < H + march_cols(T) && x < P.nx;
    const bool rows = P.walls != 0;
    const int top = P.ny - 2;  // last fluid row between walls

    MarchLevel L[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        for (int k = 0; k < 9; ++k) L[t].f[k] = 0.0;
        L[t].rho = 1.0;
        for (int k = 0; k < 3; ++k) L[t].w0[k] = L[t].w1[k] = L[t].up[k] = 0.0;
        for (int k = 0; k < 6; ++k) L[t].a[k] = 0.0;
        L[t].F[0] = L[t].F[1] = 0.0;
    }
    const int first = rows && y0 - H < 1 ? 1 : y0 - H, last = y1 + H;
    // One row of every level. f: the pulled populations of row i at level 0. WALL: some row of this
    // pass may lie next to a wall (or, with periodic rows, be stored past the seam); PART: some
    // levels may not be in use yet. A pass with neither has no condition left.
    auto row = [&](auto wall, auto part, int i, double f[9]) {
        constexpr bool WALL = decltype(wall)::value, PART = decltype(part)::value;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            MarchLevel& M = L[t];
            const int p = i - 2 * t, c = p - 1;
            // rows that collide at this level
            int lo = y0 - 2 * (T - 1 - t), hi = y1 + 2 * (T - 1 - t);
            if (rows) {
                lo = lo < 1 ? 1 : lo;
                hi = hi > top ? top : hi;
            }
            if (PART && (p < lo - 1 || (WALL && rows && p < 1))) break;  // nothing is here yet
            double n[3], rho = 1.0;
            if (!WALL || !rows || p <= top) {
                rho = sum9(f);
                n[1] = psi_of_rho<EOS>(P, rho);
                n[0] = X::left(n[1]);
                n[2] = X::right(n[1]);
                if (WALL && rows && p == 1) {  // the solid row below has this row's psi, or none
#pragma unroll
                    for (int k = 0; k < 3; ++k) M.w1[k] = P.ghost ? n[k] : 0.0;
                }
            } else {  // the solid row above
#pragma unroll
                for (int k = 0; k < 3; ++k) n[k] = P.ghost ? M.w1[k] : 0.0;
            }
            double s[9];  // f* of row c
            if ((!PART || c >= lo) && (!WALL || c <= hi)) {
#pragma unroll
                for (int k = 0; k < 9; ++k) s[k] = M.f[k];
                double sx, sy;
                cohesion_sum(M.w0[0], M.w0[1], M.w0[2], M.w1[0], M.w1[2], n[0], n[1], n[2], sx, sy);
                if constexpr (!WALL) {
                    collide_free<VISC>(P, s, M.rho, M.w1[1], sx, sy);
                } else {
                    double Ax = 0.0, Ay = 0.0;
                    if (rows && (c == 1 || c == top)) {
                        adhesion_sum(P, gw, xc, c, Ax, Ay);
                        if (GEO == GEO_WET && P.wet) {
                            if (t < T - 1)
                                total_force(P, M.rho, M.w1[1], sx, sy, Ax, Ay, M.F[0], M.F[1]);
                            else if (store)
                                store_wall_force<GEO>(P, gout, (long long)c * P.pitch + xc, P.plane,
                                                      P.pitch, c, M.rho, M.w1[1], sx, sy, Ax, Ay);
                        }
                    }
                    collide(P, s, M.rho, M.w1[1], sx, sy, Ax, Ay);
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) { M.w0[k] = M.w1[k]; M.w1[k] = n[k]; }
#pragma unroll
            for (int k = 0; k < 9; ++k) M.f[k] = f[k];
            M.rho = rho;
            if (PART && c < lo) break;
            if (t == T - 1) {
                if ((!WALL || c <= hi) && store) {
                    double* o = gout + (long long)(!WALL || rows ? c : wrapx(c, P.ny)) * P.pitch;
#pragma unroll
                    for (int k = 0; k < 9; ++k) {
                        unsigned at = 8 * xc;
                        X::opaque(at);
                        *(double*)((char*)(o + k * P.plane) + at) = s[k];
                    }
                }
            } else {
                // the next level's pull of row c - 1
                f[2] = M.a[0]; f[5] = M.a[1]; f[6] = M.a[2];
                f[0] = M.a[3]; f[1] = M.a[4]; f[3] = M.a[5];
                if (!WALL || c <= hi) {
                    f[4] = s[4];
                    f[7] = X::right(s[7]);
                    f[8] = X::left(s[8]);
                    const bool b = WALL && rows && c == 1;  // reflected at the bottom wall
                    M.a[0] = b ? s[4] : M.up[0];
                    M.a[1] = b ? s[7] : M.up[1];
                    M.a[2] = b ? s[8] : M.up[2];
                    M.a[3] = s[0];
                    M.a[4] = X::left(s[1]);
                    M.a[5] = X::right(s[3]);
                    const bool u = WALL && rows && c == top;  // kept: the top wall reflects it
                    M.up[0] = s[2];
                    M.up[1] = u ? s[5] : X::left(s[5]);
                    M.up[2] = u ? s[6] : X::right(s[6]);
                } else {  // the solid row above: row c - 1 = top is reflected
                    f[4] = M.up[0]; f[7] = M.up[1]; f[8] = M.up[2];
                }
                if (WALL && GEO == GEO_WET && P.wet) {
                    if (c == 2) wet_node_bottom(f, M.F[0], M.F[1]);
                    if (c - 1 == top) wet_node_top(f, M.F[0], M.F[1]);
                }
            }
        }
    };
    const int load_last = rows && last > top ? top : last;
    const unsigned b[3] = {8 * xc, 8 * (xc == 0 ? P.nx - 1 : xc - 1),
                           8 * (xc == (unsigned)P.nx - 1 ? 0 : xc + 1)};
    auto at = [&](int y) { return rows ? y : wrapx(y, P.ny); };
    double pf[9];  // the next row, on its way
    march_load<false, X>(P, gin, b, at(first), pf);
    // Rows up to s1 touch no wall, nor does the row after each, which is loaded meanwhile; from s0
    // on every level is in use. A segment whose first row lies clear of the bottom wall (or seam)
    // fills its levels without wall rules.
    const int s0 = rows && y0 + H < 2 * T + 2 ? 2 * T + 2 : y0 + H;
    const int lim = rows ? top - 2 : P.ny - 3;
    const int s1 = last - 1 < lim ? last - 1 : lim;
    int i = first;
    double f[9];
    const std::true_type yes;
    const std::false_type no;
    auto next = [&](int r) {  // takes the row on its way and starts the loads of row r
#pragma unroll
        for (int k = 0; k < 9; ++k) f[k] = pf[k];
        march_load<true, X>(P, gin, b, r, pf);
    };
    if (first >= 2 && s0 < s1)
        for (; i < s0; ++i) {
            next(i + 1);
            row(no, yes, i, f);
        }
    for (; i <= last; ++i) {
        if (i >= s0 && i < s1) {
            // two rows a turn, so that what one row held and what it pulled swap registers
            for (; i < s1; i += 2) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    next(i + r + 1);
                    row(no, no, i + r, f);
                }
            }
            if (i > last) break;
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) f[k] = pf[k];
        if (GEO == GEO_WET && P.wet) {
            if (i == 1) wet_node_bottom(f, gin[xc], gin[P.plane + xc]);
            const double* rt = gin + (long long)(P.ny - 1) * P.pitch;
            if (i == top) wet_node_top(f, rt[xc], rt[P.plane + xc]);
        }
        if (i < load_last) march_load<false, X>(P, gin, b, at(i + 1), pf);
        row(yes, yes, i, f);
    }
}

}  // namespace lbm
