// lbm_steps.h -- kTileSteps time steps per launch on a lattice too small to fill the GPU.
//
// What bounds such a lattice is the chain of one workgroup and the gap between dependent launches
// (about 2 us), not arithmetic: two steps per launch took 5.4-6 us however small the lattice. Here a
// launch makes four; the tile is small (8 x 4 to 16 x 8) and its halo of 8 rings recomputed, which
// costs 10 first-step updates (12.4 of psi) per node of an 8 x 4 tile on compute units that would be
// idle. One thread per node of the first region, the ring that only needs psi on waves of its own:
// every phase of a step is one psi or one collision deep on at most 11 waves. Per step, two-step
// launches and these: 120 x 60 2.70 -> 1.87 us (8 x 4), 128 x 64 2.85 -> 1.89, 160 x 80 2.80 -> 1.99 (8 x 8),
// 256 x 128 3.00 -> 2.32 (16 x 8), 300 x 102 2.84 -> 2.37. Three steps took 2.05, 2.09, 2.08, 2.33
// and 2.35.
#pragma once
#include <type_traits>
#include <utility>

#include "lbm_device.h"

namespace lbm {

// Regions of steps_tile: step k (1 .. N) updates the tile grown by 2 (N - k) rings and needs psi one
// ring further.
template <int N, int TX, int TY>
struct StepsShape {
    static constexpr int w(int k) { return TX + 4 * (N - k); }
    static constexpr int h(int k) { return TY + 4 * (N - k); }
    static constexpr int nodes(int k) { return w(k) * h(k); }
    static constexpr int ring(int k) { return 2 * (w(k) + 2) + 2 * h(k); }
};
// Threads of the workgroup: one per node of the first region, the ring around it on further waves.
constexpr int steps_threads(int N, int TX, int TY) {
    const int w = TX + 4 * (N - 1), h = TY + 4 * (N - 1);
    return ((w * h + 63) / 64 * 64 + 2 * (w + 2) + 2 * h + 63) / 64 * 64;
}

template <int N, int TX, int TY, int GEO>
struct StepsLds {
    using S = StepsShape<N, TX, TY>;
    double g1[9 * S::nodes(1)];  // populations after steps 1, 3, ...
    double g2[9 * S::nodes(2)];  // and 2, 4, ...
    double ps[(S::w(1) + 2) * (S::h(1) + 2)];
    unsigned short lk[GEO == GEO_MASK ? (S::w(1) + 2) * (S::h(1) + 2) : 1];
};

// f(1), f(2), ... f(N) with the number as a compile-time constant.
template <class F, int... K>
__device__ __forceinline__ void steps_in_turn(F&& f, std::integer_sequence<int, K...>) {
    (f(std::integral_constant<int, K + 1>{}), ...);
}

// N time steps of a TX x TY tile, by steps_threads() threads with one node each: two phases per
// step (psi of the step's region and one ring; forces and collision of the region), the
// populations between steps in LDS. The regions shrink by two rings per step. MID: the state after
// step k < N is written too, to mid + (k - 1) mstride (without the wet-node force, so not for that
// wall). The arithmetic of every node is that of step_tile: the same bits as N single steps.
template <int N, int TX, int TY, int GEO, int EOS, bool MID = false>
__device__ __forceinline__ void steps_tile(const KParams& P, const double* __restrict__ gin,
                                           double* __restrict__ gout,
                                           const double* __restrict__ gw, int x0, int y0,
                                           StepsLds<N, TX, TY, GEO>& L,
                                           double* __restrict__ mid = nullptr,
                                           long long mstride = 0) {
    static_assert(!MID || GEO == GEO_ROWS, "intermediate states carry no wet-node force");
    using S = StepsShape<N, TX, TY>;
    constexpr bool MK = GEO == GEO_MASK;
    constexpr int NT = steps_threads(N, TX, TY), LKW = S::w(1) + 2;
    const int tid = threadIdx.x;
    auto step = [&](auto kk) {
        constexpr int k = decltype(kk)::value;
        constexpr int R = 2 * (N - k), W = S::w(k), H = S::h(k), PW = W + 2;
        constexpr int WP = W + 4, PLP = WP * (H + 4);  // of the step before
        constexpr int PL = W * H, NRING = S::ring(k);
        const double* gp = k % 2 ? L.g2 : L.g1;
        double* gn = k % 2 ? L.g1 : L.g2;
        // pull behind slot (lx, ly) of the region (-1 and W, H: the ring): its populations into f;
        // false where psi is 0. fluid: a fluid node of the lattice, not a ghost row
        auto pull = [&](int lx, int ly, double f[9], bool& fluid) -> bool {
            const int gx = x0 - R + lx, gy = y0 - R + ly;
            int sx, sy;
            if constexpr (MK) {
                unsigned short& lk = L.lk[(ly + 1 + 2 * (k - 1)) * LKW + lx + 1 + 2 * (k - 1)];
                if constexpr (k == 1) {
                    sx = wrapx(gx, P.nx);
                    sy = wrapx(gy, P.ny);
                    lk = P.links[(unsigned)sy * P.pitch + sx];
                }
                const unsigned b = lk;
                fluid = !(b & 1u);
                if (!fluid) return false;
                if constexpr (k == 1) pull9_mask(P, gin, sx, sy, b, f);
                else pull9_lds_mask(gp, PLP, WP, (ly + 2) * WP + lx + 2, b, f);
                return true;
            } else {
                const bool v = slot_source(P, gx, gy, sx, sy);
                fluid = v && (!P.walls || (gy >= 1 && gy <= P.ny - 2));
                if (!v) return false;
                if constexpr (k == 1) {
                    pull9<GEO>(P, gin, sx, sy, f);
                } else {
                    // the mirrored row of a ghost slot lies next to it
                    const int row = P.walls ? sy - (y0 - R - 2) : ly + 2;
                    pull9_lds<GEO>(P, gp, PLP, WP, row * WP + lx + 2, sy, f);
                }
                return true;
            }
        };
        const int lx = tid % W, ly = tid / W;
        double f[9], rho = 1.0;
        bool ok = false;
        if (tid < PL) {
            double ps = 0.0;
            if (pull(lx, ly, f, ok)) {
                rho = sum9(f);
                ps = psi_of_rho<EOS>(P, rho);
            }
            L.ps[(ly + 1) * PW + lx + 1] = ps;
        }
        constexpr int RB = (PL + 63) / 64 * 64 + NRING <= NT ? (PL + 63) / 64 * 64 : 0;
        for (int h = tid - RB; h < NRING; h += NT) {
            if (h < 0) continue;
            int hx, hy;
            if (h < PW) { hx = h - 1; hy = -1; }
            else if (h < 2 * PW) { hx = h - PW - 1; hy = H; }
            else if (h < 2 * PW + H) { hx = -1; hy = h - 2 * PW; }
            else { hx = W; hy = h - 2 * PW - H; }
            double g[9], ps = 0.0;
            bool fluid;
            if (pull(hx, hy, g, fluid)) ps = psi_of_rho<EOS>(P, sum9(g));
            L.ps[(hy + 1) * PW + hx + 1] = ps;
        }
        __syncthreads();
        if (ok) {
            const int gx = x0 - R + lx, gy = y0 - R + ly;
            const double* c = L.ps + (ly + 1) * PW + lx + 1;
            double sx, sy, Ax = 0.0, Ay = 0.0;
            cohesion_sum(c[-PW - 1], c[-PW], c[-PW + 1], c[-1], c[1], c[PW - 1], c[PW], c[PW + 1],
                         sx, sy);
            if constexpr (MK) {
                adhesion_mask(P, wrapx(gx, P.nx), wrapx(gy, P.ny),
                              L.lk[(ly + 1 + 2 * (k - 1)) * LKW + lx + 1 + 2 * (k - 1)], Ax, Ay);
            } else {
                if (P.walls && (gy == 1 || gy == P.ny - 2))
                    adhesion_sum(P, gw, wrapx(gx, P.nx), gy, Ax, Ay);
            }
            if constexpr (k < N) {
                // a boundary node's force feeds the next step's reconstruction, which the region
                // one ring in performs; those nodes have their solid-row slot inside this one
                if (GEO == GEO_WET && P.wet && ly >= 1 && ly <= H - 2)
                    store_wall_force<GEO>(P, gn, tid, PL, W, gy, rho, c[0], sx, sy, Ax, Ay);
                collide(P, f, rho, c[0], sx, sy, Ax, Ay);
#pragma unroll
                for (int a = 0; a < 9; ++a) gn[a * PL + tid] = f[a];
                if constexpr (MID) {
                    if (lx >= R && lx < R + TX && ly >= R && ly < R + TY && gx < P.nx &&
                        gy <= P.y_hi) {
                        double* m = mid + (k - 1) * mstride + (unsigned)gy * P.pitch + gx;
#pragma unroll
                        for (int a = 0; a < 9; ++a) m[a * P.plane] = f[a];
                    }
                }
            } else if (gx < P.nx && gy <= P.y_hi) {
                const unsigned i = (unsigned)gy * P.pitch + gx;
                store_wall_force<GEO>(P, gout, i, P.plane, P.pitch, gy, rho, c[0], sx, sy, Ax, Ay);
                collide(P, f, rho, c[0], sx, sy, Ax, Ay);
#pragma unroll
                for (int a = 0; a < 9; ++a) (gout + a * P.plane)[i] = f[a];
            }
        }
        if constexpr (k < N) __syncthreads();
    };
    steps_in_turn(step, std::make_integer_sequence<int, N>{});
}

}  // namespace lbm
