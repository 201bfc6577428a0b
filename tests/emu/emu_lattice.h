// emu_lattice.h -- what the CPU emulations of the marching strips and of the multi-step tiles
// share: a seeded lattice whose slots hold NaN where they are no state, single steps of every node
// from the per-node functions alone, and the comparison, bit for bit, of every slot.
#pragma once
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <vector>

#include "../../paper_1410_2569_amd/csrc/lbm_device.h"

namespace emu {

using namespace lbm;
static const double kNaN = std::numeric_limits<double>::quiet_NaN();

static unsigned long long g_seed = 7;
static double u01() {
    g_seed = g_seed * 6364136223846793005ull + 1442695040888963407ull;
    return (double)(g_seed >> 11) * 0x1p-53;
}

struct Lattice {
    KParams P{};
    std::vector<double> g, gw;
    std::vector<unsigned short> links;
    bool fluid(int x, int y) const {
        if (P.mask) return !(links[(size_t)y * P.pitch + x] & 1u);
        return y >= P.y_lo && y <= P.y_hi;
    }
};

// A vapour with a few per cent of noise: every node differs, and stays in the EOS's domain.
static void make(Lattice& L, int nx, int ny, int walls, int ghost, int eos, int force) {
    KParams& P = L.P;
    P.nx = nx; P.ny = ny; P.walls = walls; P.ghost = ghost; P.eos = eos; P.wall_force = force;
    P.wet = walls == 2;
    P.mask = walls == 3;
    P.pitch = (nx + 31) / 32 * 32;
    P.plane = (long long)ny * P.pitch;
    const bool rows = walls == 1 || walls == 2;
    P.y_lo = rows ? 1 : 0;
    P.y_hi = rows ? ny - 2 : ny - 1;
    const double rl = eos ? 500.0 : 0.445, rv = eos ? 1.0 : 8.9e-4;
    P.RT = 0.0244618784; P.a = 0.5; P.b4 = 1.0;
    P.th_v = 0.64 / 3; P.th_m = -0.04 / 3; P.th_l = 1.0 / 3;
    P.rho1 = 1.3586; P.rho2 = 481.04;
    P.p1 = P.rho1 * P.th_v; P.p2 = P.p1 + (P.rho2 - P.rho1) * P.th_m;
    P.two_over_G = -2.0; P.negG = 1.0;
    P.s_e = P.s_z = 0.8; P.s_j = 1.0; P.s_q = 1.1;
    P.c_sig_e = P.c_sig_z = 12 * 0.1 / 0.75;
    P.h_e = P.h_z = 0.6; P.h_j = 0.5; P.h_q = 0.45;
    P.nu_v = 0.2; P.dnu = -0.1; P.s_nu_c = 1 / 1.1; P.rho_v = rv; P.inv_drho = 1 / (rl - rv);
    L.g.assign(9 * P.plane, kNaN);
    L.gw.assign((size_t)(P.mask ? ny : 2) * P.pitch, kNaN);
    if (P.mask) {  // pillars on a base row, some scattered nodes
        static const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1}, ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
        std::vector<char> solid((size_t)nx * ny);
        for (int y = 0; y < ny; ++y)
            for (int x = 0; x < nx; ++x)
                solid[(size_t)y * nx + x] = y == 0 || (y < ny / 3 && x % 7 < 3) || u01() < 0.01;
        L.links.assign(P.plane, 0xffff);
        for (int y = 0; y < ny; ++y)
            for (int x = 0; x < nx; ++x) {
                unsigned b = solid[(size_t)y * nx + x];
                for (int a = 1; a < 9; ++a)
                    if (solid[(size_t)((y - ey[a] + ny) % ny) * nx + (x - ex[a] + nx) % nx]) b |= 1u << a;
                L.links[(size_t)y * P.pitch + x] = (unsigned short)b;
            }
        P.links = L.links.data();
        P.gwn = L.gw.data();
    }
    for (int a = 0; a < 9; ++a)
        for (int y = 0; y < ny; ++y)
            for (int x = 0; x < nx; ++x)
                if (L.fluid(x, y))
                    L.g[a * P.plane + (long long)y * P.pitch + x] =
                        (a == 0 ? 4.0 / 9 : a < 5 ? 1.0 / 9 : 1.0 / 36) * rv * (1 + 0.05 * u01());
    for (int k = 0; k < (P.mask ? ny : 2); ++k)
        for (int x = 0; x < nx; ++x) L.gw[(size_t)k * P.pitch + x] = 0.01 * (u01() - 0.5);
    if (P.wet)
        for (int x = 0; x < nx; ++x)
            for (int k = 0; k < 2; ++k) {
                L.g[k * P.plane + x] = 1e-3 * rv * (u01() - 0.5);
                L.g[k * P.plane + (long long)(ny - 1) * P.pitch + x] = 1e-3 * rv * (u01() - 0.5);
            }
}

// One step of every node, from the per-node functions alone.
template <int GEO>
static void single_step(const Lattice& L, const double* gin, double* gout) {
    const KParams& P = L.P;
    for (int y = P.y_lo; y <= P.y_hi; ++y)
        for (int x = 0; x < P.nx; ++x) {
            if (!L.fluid(x, y)) continue;
            double f[9], q[3][3], sx, sy, Ax, Ay;
            pull9<GEO>(P, gin, x, y, f);
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx)
                    q[dy + 1][dx + 1] = psi_at<GEO>(P, gin, x + dx, y + dy);
            const double rho = sum9(f);
            cohesion_sum(q[0][0], q[0][1], q[0][2], q[1][0], q[1][2], q[2][0], q[2][1], q[2][2],
                         sx, sy);
            const long long i = (long long)y * P.pitch + x;
            if (P.mask) adhesion_mask(P, x, y, L.links[i], Ax, Ay);
            else adhesion_sum(P, L.gw.data(), x, y, Ax, Ay);
            store_wall_force<GEO>(P, gout, i, P.plane, P.pitch, y, rho, q[1][1], sx, sy, Ax, Ay);
            collide(P, f, rho, q[1][1], sx, sy, Ax, Ay);
            for (int a = 0; a < 9; ++a) gout[a * P.plane + i] = f[a];
        }
}

// n single steps against `out` (all NaN before the launch): every slot must hold the same bits.
template <int GEO>
static int compare(const Lattice& L, int n, const std::vector<double>& out) {
    const KParams& P = L.P;
    std::vector<double> ref = L.g;
    for (int k = 0; k < n; ++k) {
        std::vector<double> nx(ref.size(), kNaN);
        single_step<GEO>(L, ref.data(), nx.data());
        ref = nx;
    }
    int bad = 0, diff = 0;
    long long state = 0;
    for (int a = 0; a < 9; ++a)
        for (int y = 0; y < P.ny; ++y)
            for (int x = 0; x < P.nx; ++x)
                if (L.fluid(x, y)) {
                    ++state;
                    if (!std::isfinite(ref[a * P.plane + (long long)y * P.pitch + x])) ++bad;
                }
    if (bad) std::printf("the single steps are not finite at %d slots\n", bad);
    for (size_t i = 0; i < ref.size(); ++i)
        if (std::memcmp(&ref[i], &out[i], 8) && !(std::isnan(ref[i]) && std::isnan(out[i])))
            if (++diff <= 5) {
                const long long r = i % P.plane;
                std::printf("plane %lld x %lld y %lld: %.17g, single steps %.17g\n",
                            (long long)i / P.plane, r % P.pitch, r / P.pitch, out[i], ref[i]);
            }
    std::printf("%s: %d of %lld state values differ\n", diff || bad ? "FAIL" : "ok", diff, state);
    return diff || bad;
}

}  // namespace emu
