// steps_emu.cpp -- CPU emulation of the multi-step tiles of small lattices (lbm_steps.h).
//
// A workgroup is emulated by one host thread per device thread with a real barrier. Every slot that
// is not state holds NaN, the output is all NaN before the launch and the LDS before every tile, and
// the build runs under AddressSanitizer: a read of a slot that holds nothing or an access outside
// the buffers shows. The steps of one launch must equal single steps of every node bit for bit and
// leave every other slot untouched.
// Usage: steps_emu NX NY WALLS GHOST EOS FORCE TILE   (TILE: 0 8x4, 1 8x8, 2 16x8; four steps)
#include <barrier>
#include <memory>
#include <thread>

#include "emu_lattice.h"

#ifdef LBM_STEPS_HEADER
#include LBM_STEPS_HEADER
#else
#include "../../paper_1410_2569_amd/csrc/lbm_steps.h"
#endif

thread_local EmuIdx threadIdx;
static std::barrier<>* g_bar = nullptr;
void __syncthreads() { g_bar->arrive_and_wait(); }
int __syncthreads_or(int v) { return v; }

using namespace emu;

template <int TX, int TY, int GEO>
static int check(const Lattice& L) {
    constexpr int N = 4, NT = steps_threads(N, TX, TY);
    const KParams& P = L.P;
    std::vector<double> out(L.g.size(), kNaN);
    auto lds = std::make_unique<StepsLds<N, TX, TY, GEO>>();
    const int ntx = (P.nx + TX - 1) / TX, nty = (P.y_hi - P.y_lo + TY) / TY;
    std::barrier<> bar(NT);
    g_bar = &bar;
    std::vector<std::thread> th;
    for (int t = 0; t < NT; ++t)
        th.emplace_back([&, t] {
            threadIdx.x = t;
            for (int k = 0; k < ntx * nty; ++k) {
                bar.arrive_and_wait();
                if (t == 0) {
                    std::fill((double*)lds.get(), (double*)lds.get() + sizeof(*lds) / 8, kNaN);
                    for (auto& b : lds->lk) b = 0xffff;
                }
                bar.arrive_and_wait();
                steps_tile<N, TX, TY, GEO, EOS_ANY>(P, L.g.data(), out.data(), L.gw.data(),
                                                    k % ntx * TX, P.y_lo + k / ntx * TY, *lds);
            }
        });
    for (auto& t : th) t.join();
    return compare<GEO>(L, N, out);
}

template <int GEO>
static int check(const Lattice& L, int tile) {
    return tile == 0 ? check<8, 4, GEO>(L) : tile == 1 ? check<8, 8, GEO>(L) : check<16, 8, GEO>(L);
}

int main(int argc, char** argv) {
    if (argc != 8) return 2;
    int v[7];
    for (int k = 0; k < 7; ++k) v[k] = std::atoi(argv[k + 1]);
    Lattice L;
    make(L, v[0], v[1], v[2], v[3], v[4], v[5]);
    if (L.P.mask) return check<GEO_MASK>(L, v[6]);
    return L.P.wet ? check<GEO_WET>(L, v[6]) : check<GEO_ROWS>(L, v[6]);
}
