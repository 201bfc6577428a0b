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
#include <thread>

#include "emu_lattice.h"

#ifdef LBM_MARCH_HEADER
#include LBM_MARCH_HEADER
#else
#include "../../paper_1410_2569_amd/csrc/lbm_march.h"
#endif

thread_local EmuIdx threadIdx;
void __syncthreads() {}
int __syncthreads_or(int v) { return v; }

using namespace emu;
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
static int check(const Lattice& L, int T, int h) {
    std::vector<double> out(L.g.size(), kNaN);
    if (T == 2) march<2, GEO>(L.P, L.g.data(), out.data(), L.gw.data(), h);
    else if (T == 3) march<3, GEO>(L.P, L.g.data(), out.data(), L.gw.data(), h);
    else march<4, GEO>(L.P, L.g.data(), out.data(), L.gw.data(), h);
    return compare<GEO>(L, T, out);
}

int main(int argc, char** argv) {
    if (argc != 9) return 2;
    int v[8];
    for (int k = 0; k < 8; ++k) v[k] = std::atoi(argv[k + 1]);
    g_lane[0] = g_lane[65] = kNaN;
    Lattice L;
    make(L, v[0], v[1], v[2], v[3], v[4], v[5]);
    return L.P.wet ? check<GEO_WET>(L, v[6], v[7]) : check<GEO_ROWS>(L, v[6], v[7]);
}
