// obs_emu.cpp -- CPU emulation of the observables' tiles and final sums (lbm_obs.h).
//
// A workgroup is emulated by one host thread per device thread with real barriers, its wave-wide
// votes and exchanges by barriers of 64 threads. Every slot that is not state holds NaN, the partial
// rows are all NaN before the launch and the LDS before every tile, and the build runs under
// AddressSanitizer. Every partial row must equal, bit for bit, the tree over obs_node's values of
// its 64 x 4 nodes (psi and density from psi_node, through fields of the lattice), every row must be
// written, and the final block must give the sums of the rows in its stated order.
// Usage: obs_emu NX NY WALLS GHOST EOS FORCE PRE ROWS   (ROWS: 4 or 8 per block)
#include <barrier>
#include <memory>
#include <thread>

#include "emu_lattice.h"

thread_local EmuIdx threadIdx;
static std::barrier<> g_bar(256);
static std::barrier<> g_wave[4] = {std::barrier<>(64), std::barrier<>(64), std::barrier<>(64),
                                   std::barrier<>(64)};
void __syncthreads() { g_bar.arrive_and_wait(); }
int __syncthreads_or(int v) { return v; }
// What the lanes of a wave show each other, in two places by turns: a lane that has passed the
// barrier may write its next value while another still reads this one.
static double g_slot[2][256];
static const double* shown(double v) {
    static thread_local int turn = 0;
    const unsigned t = threadIdx.x;
    turn ^= 1;
    g_slot[turn][t] = v;
    g_wave[t / 64].arrive_and_wait();
    return g_slot[turn];
}
static double __shfl_xor(double v, int mask, int) { return shown(v)[threadIdx.x ^ mask]; }
static int __any(int v) {
    const double* s = shown(v) + threadIdx.x / 64 * 64;
    int r = 0;
    for (int k = 0; k < 64; ++k) r |= s[k] != 0;
    return r;
}

#ifdef LBM_OBS_HEADER
#include LBM_OBS_HEADER
#else
#include "../../paper_1410_2569_amd/csrc/lbm_obs.h"
#endif

using namespace emu;

// One workgroup of 256 threads runs `body` n times.
template <class F>
static void workgroup(int n, F&& body) {
    std::vector<std::thread> th;
    for (int t = 0; t < 256; ++t)
        th.emplace_back([&, t] {
            threadIdx.x = t;
            for (int k = 0; k < n; ++k) body(k);
        });
    for (auto& t : th) t.join();
}

static int differ(const std::vector<double>& got, const std::vector<double>& want, const char* what) {
    int n = 0;
    for (size_t i = 0; i < want.size(); ++i)
        if (std::memcmp(&got[i], &want[i], 8) && !(std::isnan(got[i]) && std::isnan(want[i])))
            if (++n <= 5)
                std::printf("%s: row %zu quantity %zu: %.17g, expected %.17g\n", what, i / O_NQ,
                            i % O_NQ, got[i], want[i]);
    return n;
}

// Partial rows from obs_node: per wave the exchange tree's sum, then the four waves.
template <bool PRE>
static std::vector<double> rows_by_node(const Lattice& L, const double* g, const ObsArgs& A) {
    const KParams& P = L.P;
    std::vector<double> psi(P.plane, kNaN), rho(P.plane, kNaN);
    if (P.walls && !P.mask && !P.ghost)
        for (int x = 0; x < P.nx; ++x) psi[x] = psi[(size_t)(P.ny - 1) * P.pitch + x] = 0.0;
    for (int y = P.y_lo; y <= P.y_hi; ++y)
        for (int x = 0; x < P.nx; ++x) psi_node<PRE>(P, g, psi.data(), rho.data(), x, y);
    const int nbx = (P.nx + 63) / 64, n = obs_rows(P);
    std::vector<double> out((size_t)n * O_NQ);
    for (int b = 0; b < n; ++b)
        for (int q = 0; q < O_NQ; ++q) {
            double w[4];
            for (int r = 0; r < 4; ++r) {
                double s[64];
                for (int l = 0; l < 64; ++l) {
                    const int x = b % nbx * 64 + l, y = P.y_lo + b / nbx * 4 + r;
                    double v[O_NQ];
                    for (int k = 0; k < O_NQ; ++k) v[k] = op_identity(k);
                    if (x < P.nx && y <= P.y_hi)
                        obs_node<PRE>(P, g, rho.data(), psi.data(), L.gw.data(), A, x, y, v);
                    s[l] = v[q];
                }
                for (int off = 32; off > 0; off >>= 1)
                    for (int l = 0; l < off; ++l) s[l] = op_combine(q, s[l], s[l + off]);
                w[r] = s[0];
            }
            out[(size_t)b * O_NQ + q] = op_combine(q, op_combine(q, w[0], w[1]),
                                                   op_combine(q, w[2], w[3]));
        }
    return out;
}

static std::vector<double> final_by_order(const std::vector<double>& part, int n) {
    std::vector<double> out(O_NQ);
    for (int q = 0; q < O_NQ; ++q) {
        double s[256];
        for (int t = 0; t < 256; ++t) {
            s[t] = op_identity(q);
            for (int b = t; b < n; b += 256) s[t] = op_combine(q, s[t], part[(size_t)b * O_NQ + q]);
        }
        for (int w = 128; w > 0; w >>= 1)
            for (int t = 0; t < w; ++t) s[t] = op_combine(q, s[t], s[t + w]);
        out[q] = s[0];
    }
    return out;
}

static int check_final(const std::vector<double>& part, int n) {
    static double sh[O_NQ][256];
    std::fill(&sh[0][0], &sh[0][0] + O_NQ * 256, kNaN);
    std::vector<double> out(O_NQ, kNaN);
    workgroup(1, [&](int) { obs_final_block(part.data(), n, sh, out.data()); });
    return differ(out, final_by_order(part, n), "final");
}

template <bool PRE, int ROWS>
static int check(const Lattice& L, const ObsArgs& A, const char* what) {
    const KParams& P = L.P;
    std::vector<double> g = L.g;
    if (PRE)  // the caller holds pre-collision populations; solid nodes hold nothing
        for (int y = P.y_lo; y <= P.y_hi; ++y)
            for (int x = 0; x < P.nx; ++x) {
                if (!L.fluid(x, y)) continue;
                double f[9];
                pull9_any(P, L.g.data(), x, y, f);
                for (int a = 0; a < 9; ++a) g[a * P.plane + (long long)y * P.pitch + x] = f[a];
            }
    const int nbx = (P.nx + 63) / 64, nby = (P.y_hi - P.y_lo + ROWS) / ROWS;
    std::vector<double> part((size_t)obs_rows(P) * O_NQ, kNaN);
    auto lds = std::make_unique<ObsLds<ROWS>>();
    workgroup(nbx * nby, [&](int k) {
        g_bar.arrive_and_wait();
        if (threadIdx.x == 0)
            std::fill((double*)lds.get(), (double*)lds.get() + sizeof(*lds) / 8, kNaN);
        g_bar.arrive_and_wait();
        obs_tile<PRE, ROWS>(P, g.data(), L.gw.data(), A, k % nbx, k / nbx, nbx, part.data(), *lds);
    });
    const std::vector<double> want = rows_by_node<PRE>(L, g.data(), A);
    double points = 0.0, bad = 0.0;
    for (size_t b = 0; b < want.size() / O_NQ; ++b) {
        points += want[b * O_NQ + O_N];
        bad += want[b * O_NQ + O_BAD];
    }
    const int n = differ(part, want, what) + check_final(part, obs_rows(P));
    std::printf("%s: %s, %d of %zu differ; %g interface points, %g nodes not finite\n", what,
                n ? "FAIL" : "ok", n, want.size(), points, bad);
    return n;
}

template <bool PRE, int ROWS>
static int check_all(Lattice& L) {
    const KParams& P = L.P;
    const double yw = P.wet ? 1.0 : 0.5, inf = __builtin_huge_val();
    const double mid = 1.025 * P.rho_v;  // the noise crosses it at every other edge
    int n = check<PRE, ROWS>(L, {mid, yw + 3.0, -inf, inf, 0.5 * P.nx, yw}, "all edges");
    n += check<PRE, ROWS>(L, {mid, 2.0, 0.25 * P.nx, 0.6 * P.nx, 0.4 * P.nx, 2.0}, "a window");
    // nodes that are no numbers, in the first rows and at the far corner: without edges in their
    // waves, then with
    for (int k = 0; k < 2; ++k) {
        const int x = k ? P.nx - 1 : P.nx / 2, y = k ? P.y_hi : P.y_lo;
        if (L.fluid(x, y)) L.g[(long long)y * P.pitch + x] = kNaN;
    }
    n += check<PRE, ROWS>(L, {10.0 * P.rho_v, yw, -inf, inf, 0.5 * P.nx, yw}, "not finite, no edge");
    n += check<PRE, ROWS>(L, {mid, yw, -inf, inf, 0.5 * P.nx, yw}, "not finite");
    return n;
}

int main(int argc, char** argv) {
    if (argc != 9) return 2;
    int v[8];
    for (int k = 0; k < 8; ++k) v[k] = std::atoi(argv[k + 1]);
    Lattice L;
    make(L, v[0], v[1], v[2], v[3], v[4], v[5]);
    int n = v[7] == 4 ? (v[6] ? check_all<true, 4>(L) : check_all<false, 4>(L))
                      : (v[6] ? check_all<true, 8>(L) : check_all<false, 8>(L));
    for (int rows : {1, 256, 700}) {  // the final block over more rows than threads
        std::vector<double> part((size_t)rows * O_NQ);
        for (double& p : part) p = u01() - 0.5;
        n += check_final(part, rows);
    }
    std::printf("%s\n", n ? "FAIL" : "ok: 0 differ");
    return n != 0;
}
