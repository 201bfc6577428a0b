// march_emu.cpp -- CPU emulation of the register-marching strips (lbm_march.h).
//
// A wave is emulated by 64 host threads in lock step; its cross-lane moves go through an array
// between two barriers. Every slot that is not state holds NaN and the output is all NaN before the
// launch, lanes past the ends of the wave shift in NaN, and the build runs under AddressSanitizer:
// a read of a slot that holds nothing, an access outside the buffers or a lane used outside its
// valid range shows. The T steps of one launch must equal T single steps of every node bit for bit
// and leave every other slot untouched.
// Usage: march_emu NX NY WALLS GHOST EOS FORCE T H   (H: rows per segment)
#include <barrier>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <thread>
#include <vector>

#ifdef LBM_MARCH_HEADER
#include LBM_MARCH_HEADER
#else
#include "../../paper_1410_2569_amd/csrc/lbm_march.h"
#endif

thread_local EmuIdx threadIdx;
void __syncthreads() {}
int __syncthreads_or(int v) { return v; }

using namespace lbm;
static const double kNaN = std::numeric_limits<double>::quiet_NaN();
static std::barrier<> g_bar(64);
static double g_lane[66];

struct EmuLane {
    static double at(double v, int d) {
        const int l = threadIdx.x;
        g_lane[l + 1] = v;
        g_bar.arrive_and_wait();
        const double r = g_lane[l + 1 + d];
        g_bar.arrive_and_wait();
        return r;
    }
    static void opaque(unsigned&) {}
    static double left(double v) { return at(v, -1); }
    static double right(double v) { return at(v, 1); }
};

static unsigned long long g_seed = 7;
static double u01() {
    g_seed = g_seed * 6364136223846793005ull + 1442695040888963407ull;
    return (double)(g_seed >> 11) * 0x1p-53;
}

static bool fluid_row(const KParams& P, int y) { return y >= P.y_lo && y <= P.y_hi; }

// One step of every node, from the per-node functions alone.
template <int GEO>
static void single_step(const KParams& P, const double* gin, double* gout, const double* gw) {
    for (int y = P.y_lo; y <= P.y_hi; ++y)
        for (int x = 0; x < P.nx; ++x) {
            double f[9], q[3][3], sx, sy, Ax, Ay;
            pull9<GEO>(P, gin, x, y, f);
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx)
                    q[dy + 1][dx + 1] = psi_at<GEO>(P, gin, x + dx, y + dy);
            const double rho = sum9(f);
            cohesion_sum(q[0][0], q[0][1], q[0][2], q[1][0], q[1][2], q[2][0], q[2][1], q[2][2],
                         sx, sy);
            adhesion_sum(P, gw, x, y, Ax, Ay);
            const long long i = (long long)y * P.pitch + x;
            store_wall_force<GEO>(P, gout, i, P.plane, P.pitch, y, rho, q[1][1], sx, sy, Ax, Ay);
            collide(P, f, rho, q[1][1], sx, sy, Ax, Ay);
            for (int a = 0; a < 9; ++a) gout[a * P.plane + i] = f[a];
        }
}

template <int T, int GEO>
static void march(const KParams& P, const double* gin, double* gout, const double* gw, int h) {
    const int nstrips = (P.nx + march_cols(T) - 1) / march_cols(T);
    std::vector<std::thread> th;
    for (int l = 0; l < 64; ++l)
        th.emplace_back([&, l] {
            threadIdx.x = l;
            for (int y0 = P.y_lo; y0 <= P.y_hi; y0 += h)
                for (int s = 0; s < nstrips; ++s) {
                    const int y1 = y0 + h - 1 < P.y_hi ? y0 + h - 1 : P.y_hi;
                    march_strip<T, GEO, EOS_ANY, 2, EmuLane>(P, gin, gout, gw, s * march_cols(T), y0,
                                                          y1, l);
                }
        });
    for (auto& t : th) t.join();
}

template <int GEO>
static int check(const KParams& P, const std::vector<double>& g0, const double* gw, int T, int h) {
    const size_t n = g0.size();
    std::vector<double> ref = g0, out(n, kNaN);
    for (int k = 0; k < T; ++k) {
        std::vector<double> nx(n, kNaN);
        single_step<GEO>(P, ref.data(), nx.data(), gw);
        ref = nx;
    }
    if (T == 2) march<2, GEO>(P, g0.data(), out.data(), gw, h);
    else if (T == 3) march<3, GEO>(P, g0.data(), out.data(), gw, h);
    else march<4, GEO>(P, g0.data(), out.data(), gw, h);
    int bad = 0;
    long long state = 0;
    for (int a = 0; a < 9; ++a)
        for (int y = 0; y < P.ny; ++y)
            for (int x = 0; x < P.nx; ++x)
                if (fluid_row(P, y)) {
                    ++state;
                    if (!std::isfinite(ref[a * P.plane + (long long)y * P.pitch + x])) ++bad;
                }
    if (bad) std::printf("the single steps are not finite at %d slots\n", bad);
    int diff = 0;
    for (size_t i = 0; i < n; ++i)
        if (std::memcmp(&ref[i], &out[i], 8) && !(std::isnan(ref[i]) && std::isnan(out[i])))
            if (++diff <= 5) {
                const long long r = i % P.plane;
                std::printf("plane %lld x %lld y %lld: %.17g, single steps %.17g\n",
                            (long long)i / P.plane, r % P.pitch, r / P.pitch, out[i], ref[i]);
            }
    std::printf("%s: %d of %lld state values differ\n", diff || bad ? "FAIL" : "ok", diff, state);
    return diff || bad;
}

int main(int argc, char** argv) {
    if (argc != 9) return 2;
    int v[8];
    for (int k = 0; k < 8; ++k) v[k] = std::atoi(argv[k + 1]);
    g_lane[0] = g_lane[65] = kNaN;
    KParams P{};
    P.nx = v[0]; P.ny = v[1]; P.walls = v[2]; P.ghost = v[3]; P.eos = v[4]; P.wall_force = v[5];
    P.wet = P.walls == 2;
    P.pitch = (P.nx + 31) / 32 * 32;
    P.plane = (long long)P.ny * P.pitch;
    P.y_lo = P.walls ? 1 : 0;
    P.y_hi = P.walls ? P.ny - 2 : P.ny - 1;
    const double rl = P.eos ? 500.0 : 0.445, rv = P.eos ? 1.0 : 8.9e-4;
    P.RT = 0.0244618784; P.a = 0.5; P.b4 = 1.0;
    P.th_v = 0.64 / 3; P.th_m = -0.04 / 3; P.th_l = 1.0 / 3;
    P.rho1 = 1.3586; P.rho2 = 481.04;
    P.p1 = P.rho1 * P.th_v; P.p2 = P.p1 + (P.rho2 - P.rho1) * P.th_m;
    P.two_over_G = -2.0; P.negG = 1.0;
    P.s_e = P.s_z = 0.8; P.s_j = 1.0; P.s_q = 1.1;
    P.c_sig_e = P.c_sig_z = 12 * 0.1 / 0.75;
    P.h_e = P.h_z = 0.6; P.h_j = 0.5; P.h_q = 0.45;
    P.nu_v = 0.2; P.dnu = -0.1; P.s_nu_c = 1 / 1.1; P.rho_v = rv; P.inv_drho = 1 / (rl - rv);
    // a vapour with a few per cent of noise: every node differs, and stays in the EOS's domain
    std::vector<double> g(9 * P.plane, kNaN), gw(2 * P.pitch, kNaN);
    for (int a = 0; a < 9; ++a)
        for (int y = P.y_lo; y <= P.y_hi; ++y)
            for (int x = 0; x < P.nx; ++x)
                g[a * P.plane + (long long)y * P.pitch + x] =
                    (a == 0 ? 4.0 / 9 : a < 5 ? 1.0 / 9 : 1.0 / 36) * rv * (1 + 0.05 * u01());
    for (int x = 0; x < P.nx; ++x)
        for (int k = 0; k < 2; ++k) gw[k * P.pitch + x] = 0.01 * (u01() - 0.5);
    if (P.wet)
        for (int x = 0; x < P.nx; ++x)
            for (int k = 0; k < 2; ++k) {
                g[k * P.plane + x] = 1e-3 * rv * (u01() - 0.5);
                g[k * P.plane + (long long)(P.ny - 1) * P.pitch + x] = 1e-3 * rv * (u01() - 0.5);
            }
    return P.wet ? check<GEO_WET>(P, g, gw.data(), v[6], v[7])
                 : check<GEO_ROWS>(P, g, gw.data(), v[6], v[7]);
}
