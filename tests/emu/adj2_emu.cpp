// adj2_emu.cpp -- CPU emulation of the two-reverse-steps tile (lbm_adj2.h) against two single
// reverse steps (adj_tile, checked by tile_emu.cpp): workgroups on host threads with a real barrier,
// NaN in every slot that is not written state and in the LDS before each tile, AddressSanitizer on.
// Every output, the wall gradient included, must hold the same bits, every other slot NaN.
// Usage: adj2_emu NX NY WALLS GHOST EOS FORCE
#include <barrier>
#include <functional>
#include <memory>
#include <thread>

#include "emu_lattice.h"

#ifdef LBM_ADJ2_HEADER
#include LBM_ADJ2_HEADER
#else
#include "../../paper_1410_2569_amd/csrc/lbm_adj2.h"
#endif

thread_local EmuIdx threadIdx;
static std::barrier<>* g_bar = nullptr;
void __syncthreads() { g_bar->arrive_and_wait(); }
int __syncthreads_or(int v) { return v; }

using namespace emu;

// Runs fn(tile) for every tile on nt threads, with `poison` between tiles.
static void groups(int nt, int ntiles, const std::function<void()>& poison,
                   const std::function<void(int)>& fn) {
    std::barrier<> bar(nt);
    g_bar = &bar;
    std::vector<std::thread> th;
    for (int t = 0; t < nt; ++t)
        th.emplace_back([&, t] {
            threadIdx.x = t;
            for (int k = 0; k < ntiles; ++k) {
                bar.arrive_and_wait();
                if (t == 0) poison();
                bar.arrive_and_wait();
                fn(k);
                // threads that have left the tile early take no further barrier of it
            }
            bar.arrive_and_drop();
        });
    for (auto& t : th) t.join();
}

struct Set {  // one step's adjoint quantities
    std::vector<double> a, q, p0, dpsi, rv;
    explicit Set(const KParams& P)
        : a(9 * P.plane, kNaN), q(2 * P.plane, kNaN), p0(P.plane, kNaN), dpsi(P.plane, kNaN),
          rv(4 * P.pitch, kNaN) {}
};

static AdjPtrs ptrs(const double* g, Set& in, Set& out, const double* gw, double* gg) {
    return {g, in.a.data(), in.q.data(), in.p0.data(), in.dpsi.data(), in.rv.data(), gw,
            out.a.data(), out.q.data(), out.p0.data(), out.dpsi.data(), out.rv.data(), gg};
}

int main(int argc, char** argv) {
    if (argc != 7) return 2;
    int v[6];
    for (int k = 0; k < 6; ++k) v[k] = std::atoi(argv[k + 1]);
    Lattice L;
    make(L, v[0], v[1], v[2], v[3], v[4], v[5]);
    const KParams& P = L.P;
    std::vector<double> g2 = L.g, g1(g2.size(), kNaN);  // the earlier and the later forward state
    single_step<GEO_ROWS>(L, g2.data(), g1.data());
    Set in(P), mid(P), ref(P), out(P);
    auto fill = [&](std::vector<double>& f, int planes) {
        for (int a = 0; a < planes; ++a)
            for (int y = P.y_lo; y <= P.y_hi; ++y)
                for (int x = 0; x < P.nx; ++x) f[a * P.plane + (long long)y * P.pitch + x] = u01() - 0.5;
    };
    fill(in.a, 9);
    fill(in.q, 2);
    fill(in.p0, 1);
    fill(in.dpsi, 1);
    for (int k = 0; k < 4; ++k)
        for (int x = 0; x < P.nx; ++x) in.rv[k * P.pitch + x] = u01() - 0.5;
    std::vector<double> gg(2 * P.pitch, kNaN);
    for (int k = 0; k < 2; ++k)
        for (int x = 0; x < P.nx; ++x) gg[k * P.pitch + x] = u01() - 0.5;
    std::vector<double> gg2 = gg;
    auto poison = [](auto& lds) {
        std::fill((double*)&lds, (double*)&lds + sizeof(lds) / 8, kNaN);
    };
    {
        AdjLds<32, 4> lds;
        const int ntx = (P.nx + 31) / 32, nty = (P.y_hi - P.y_lo + 4) / 4;
        auto one = [&](const AdjPtrs& A) {
            groups(128, ntx * nty, [&] { poison(lds); }, [&](int k) {
                adj_tile<32, 4, 128, EOS_ANY>(P, A, k % ntx * 32, P.y_lo + k / ntx * 4, lds);
            });
        };
        one(ptrs(g1.data(), in, mid, L.gw.data(), gg.data()));
        one(ptrs(g2.data(), mid, ref, L.gw.data(), gg.data()));
    }
    {
        auto lds = std::make_unique<Adj2Lds>();
        const int ntx = (P.nx + kAdj2X - 1) / kAdj2X, nty = (P.y_hi - P.y_lo + kAdj2Y) / kAdj2Y;
        const Adj2Ptrs B{ptrs(g1.data(), in, out, L.gw.data(), gg2.data()), g2.data()};
        groups(kAdj2Threads, ntx * nty, [&] { poison(*lds); }, [&](int k) {
            adj2_tile<EOS_ANY>(P, B, k % ntx * kAdj2X, P.y_lo + k / ntx * kAdj2Y, *lds);
        });
    }
    int diff = 0, live = 0;
    auto same = [&](const char* what, const std::vector<double>& r, const std::vector<double>& o) {
        for (size_t i = 0; i < r.size(); ++i) {
            live += !std::isnan(r[i]);
            if (std::memcmp(&r[i], &o[i], 8) && !(std::isnan(r[i]) && std::isnan(o[i])))
                if (++diff <= 6)
                    std::printf("%s %zu: %.17g, single steps %.17g\n", what, i, o[i], r[i]);
        }
    };
    same("a", ref.a, out.a);
    same("q", ref.q, out.q);
    same("p0", ref.p0, out.p0);
    same("dpsi", ref.dpsi, out.dpsi);
    same("rv", ref.rv, out.rv);
    same("grad", gg, gg2);
    const int want = 13 * P.nx * (P.y_hi - P.y_lo + 1) + (P.walls ? 4 * P.nx : 0) + 2 * P.nx;
    std::printf("%s: %d differ of %d (%d expected)\n", diff || live != want ? "FAIL" : "ok", diff, live, want);
    return diff || live != want;
}
