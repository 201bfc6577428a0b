// lbm_adj2.h -- two reverse steps per launch on a lattice too small to fill the GPU.
//
// What bounds the reverse sweep of such a lattice is launches: about 6.2 us of dependent launch on
// the device and 5 us on the host each, for 1.4 us of arithmetic chain. Two steps per launch share
// one launch, one round trip to memory and the stores of the step in between, whose quantities stay
// in LDS; the first step is recomputed on two rings around the tile, which costs compute units that
// would wait.
#pragma once
#include "lbm_device.h"

namespace lbm {

// Two reverse steps: of the later one, whose forward state is gprev, and of the one before it, whose
// forward state is gprev2.
struct Adj2Ptrs {
    AdjPtrs A;             // gprev and the adjoint quantities in and out
    const double* gprev2;
};

constexpr int kAdj2X = 16, kAdj2Y = 8;      // tile
constexpr int kAdj2W = kAdj2X + 4, kAdj2H = kAdj2Y + 4;  // the first step's region: two rings
// 240 threads for its nodes (4 waves), 128 for the tile's (2 waves), a wave for psi of the ring
constexpr int kAdj2First = 256, kAdj2Threads = kAdj2First + kAdj2X * kAdj2Y + 64;

struct Adj2Lds {
    static constexpr int W1 = kAdj2X + 2, H1 = kAdj2Y + 2;   // tile and one ring
    static constexpr int W2 = kAdj2W, H2 = kAdj2H;           // two rings
    static constexpr int W3 = kAdj2X + 6, H3 = kAdj2Y + 6;   // three
    static constexpr int W4 = kAdj2X + 8, H4 = kAdj2Y + 8;   // four
    double sp1[W3 * H3];               // psi of gprev
    double sp2[W1 * H1];               // psi of gprev2
    double qx[W4 * H4], qy[W4 * H4];   // q of the step after the first
    double c0[W3 * H3];                // its c
    double a1[9][W1 * H1];             // the first step's a, q, c
    double q1x[W2 * H2], q1y[W2 * H2];
    double c1[W1 * H1];
    double rv1[4][W2];                 // its wall vectors (bottom x, y; top x, y)
};

// lambda gathered at LDS slot l (row stride W) of a and c: the transposed streaming, as
// push_gather_a and push_add_c make it from memory.
__device__ __forceinline__ void push_gather_lds(const KParams& P, const double (*a)[Adj2Lds::W1 * Adj2Lds::H1],
                                                const double* c, int W, int l, int y,
                                                double nu[9]) {
    const bool bot = P.walls && y == 1, top = P.walls && y == P.ny - 2;
    const int up = top ? 0 : W, dn = bot ? 0 : W, sx = 1;
    // where a population would travel into the wall, its reflection stays on the node
    const int l2 = l + up, l5 = top ? l : l + W + sx, l6 = top ? l : l + W - sx;
    const int l4 = l - dn, l7 = bot ? l : l - W - sx, l8 = bot ? l : l - W + sx;
    nu[0] = a[0][l] + c[l];
    nu[1] = a[1][l + 1] + c[l + 1];
    nu[3] = a[3][l - 1] + c[l - 1];
    nu[2] = (top ? a[4][l2] : a[2][l2]) + c[l2];
    nu[5] = (top ? a[7][l5] : a[5][l5]) + c[l5];
    nu[6] = (top ? a[8][l6] : a[6][l6]) + c[l6];
    nu[4] = (bot ? a[2][l4] : a[4][l4]) + c[l4];
    nu[7] = (bot ? a[5][l7] : a[7][l7]) + c[l7];
    nu[8] = (bot ? a[6][l8] : a[8][l8]) + c[l8];
}

// Two reverse steps of a kAdj2X x kAdj2Y tile at (x0, y0), by kAdj2Threads threads; bounce-back or
// periodic rows. Every node's arithmetic is that of adj_tile_impl, in its order: the same bits as
// two single reverse steps. dL/dG_w receives the wall vectors of the step after the first, then the
// first step's; the second's go out.
template <int EOS>
__device__ __forceinline__ void adj2_tile(const KParams& P, const Adj2Ptrs& B, int x0, int y0,
                                          Adj2Lds& L) {
#pragma clang fp contract(off)
    using S = Adj2Lds;
    constexpr int W1 = S::W1, H1 = S::H1, W2 = S::W2, H2 = S::H2, W3 = S::W3, H3 = S::H3,
                  W4 = S::W4, H4 = S::H4, NT = kAdj2Threads, N2 = W2 * H2;
    const AdjPtrs& A = B.A;
    const int tid = threadIdx.x;
    // lattice node of a position: columns wrap, rows wrap or must be fluid rows
    auto node = [&](int gx, int gy, int& sx, int& sy) {
        sx = wrapx(gx, P.nx);
        sy = P.walls ? gy : wrapx(gy, P.ny);
        return !P.walls || (gy >= 1 && gy <= P.ny - 2);
    };

    // ---- every load of memory ----
    // first step: threads [0, 240) own a node of the region; second: [256, 384) one of the tile
    const int t2 = tid - kAdj2First;
    const bool first = tid < N2, second = t2 >= 0 && t2 < kAdj2X * kAdj2Y;
    const int lx = first ? tid % W2 : t2 % kAdj2X, ly = first ? tid / W2 : t2 / kAdj2X;
    const int gx = first ? x0 - 2 + lx : x0 + lx, gy = first ? y0 - 2 + ly : y0 + ly;
    int x = 0, y = 0;
    bool act = (first || second) && node(gx, gy, x, y);
    if (second) act = act && gx < P.nx && gy <= P.y_hi;
    double f[9], rho = 1.0, psi_c = 0.0, av[9], Ax = 0.0, Ay = 0.0;
    const bool wall_row = act && P.walls && (y == 1 || y == P.ny - 2);
    if (act) {
        pull9<GEO_ROWS>(P, first ? A.gprev : B.gprev2, x, y, f);
        rho = sum9(f);
        psi_c = psi_of_rho<EOS>(P, rho);
        if (first) push_gather_a(P, A.a_in, x, y, av);
        if (wall_row) adhesion_sum(P, A.gw, x, y, Ax, Ay);
    }
    if (first) L.sp1[(ly + 1) * W3 + lx + 1] = act ? psi_c : psi_at<GEO_ROWS, EOS>(P, A.gprev, gx, gy);
    if (second)
        L.sp2[(ly + 1) * W1 + lx + 1] = act ? psi_c : psi_at<GEO_ROWS, EOS>(P, B.gprev2, gx, gy);
    // psi of the rings: gprev's around the region (threads 256 on), gprev2's around the tile (the
    // last wave)
    auto ring = [](int h, int w, int hh, int& rx, int& ry) {  // slot h of the ring around w x hh
        if (h < w + 2) { rx = h - 1; ry = -1; }
        else if (h < 2 * (w + 2)) { rx = h - (w + 2) - 1; ry = hh; }
        else if (h < 2 * (w + 2) + hh) { rx = -1; ry = h - 2 * (w + 2); }
        else { rx = w; ry = h - 2 * (w + 2) - hh; }
    };
    if (t2 >= 0 && t2 < 2 * (W2 + 2) + 2 * H2) {
        int rx, ry;
        ring(t2, W2, H2, rx, ry);
        L.sp1[(ry + 1) * W3 + rx + 1] = psi_at<GEO_ROWS, EOS>(P, A.gprev, x0 - 2 + rx, y0 - 2 + ry);
    }
    const int t3 = t2 - kAdj2X * kAdj2Y;
    if (t3 >= 0 && t3 < 2 * W1 + 2 * kAdj2Y) {
        int rx, ry;
        ring(t3, kAdj2X, kAdj2Y, rx, ry);
        L.sp2[(ry + 1) * W1 + rx + 1] = psi_at<GEO_ROWS, EOS>(P, B.gprev2, x0 + rx, y0 + ry);
    }
    // q on four rings (0 outside the fluid rows); p0 and psi' on three
    for (int s = tid; s < W4 * H4; s += NT) {
        int sx, sy;
        double vx = 0.0, vy = 0.0;
        if (node(x0 - 4 + s % W4, y0 - 4 + s / W4, sx, sy)) {
            const unsigned i = (unsigned)sy * P.pitch + sx;
            vx = A.q_in[i];
            vy = (A.q_in + P.plane)[i];
        }
        L.qx[s] = vx;
        L.qy[s] = vy;
    }
    const int cx = tid % W3, cy = tid / W3;
    const bool has_c = tid < W3 * H3;
    int ccx, ccy = 0;
    const bool fluid_c = has_c && node(x0 - 3 + cx, y0 - 3 + cy, ccx, ccy);
    double p0v = 0.0, dpv = 0.0;
    if (fluid_c) {
        const unsigned i = (unsigned)ccy * P.pitch + ccx;
        p0v = A.p0_in[i];
        dpv = A.dpsi_in[i];
    }
    __syncthreads();
    // ---- c of the step after the first, on three rings (0 on solid rows) ----
    if (has_c)
        L.c0[tid] = fluid_c ? dpv * adj_xi(P, L.qx, L.qy, W4, (cy + 1) * W4 + cx + 1, ccy, p0v) : 0.0;
    __syncthreads();

    // ---- the first step on two rings ----
    double p01 = 0.0, dpsi1 = 0.0;
    const bool in1 = first && lx >= 1 && lx < W2 - 1 && ly >= 1 && ly < H2 - 1;  // one ring
    const int l1 = (ly - 1) * W1 + lx - 1;
    if (first) {
        double qx = 0.0, qy = 0.0;
        if (act) {
            const int l3 = (ly + 1) * W3 + lx + 1;
            const double* cc = L.sp1 + l3;
            double sx, sy, nu[9], fb[9], rx, ry;
            cohesion_sum(cc[-W3 - 1], cc[-W3], cc[-W3 + 1], cc[-1], cc[1], cc[W3 - 1], cc[W3],
                         cc[W3 + 1], sx, sy);
            push_add_c(P, av, L.c0, W3, l3, y, nu);
            collide_adj(P, f, rho, psi_c, sx, sy, Ax, Ay, nu, fb, p01, qx, qy, rx, ry);
            dpsi1 = dpsi_drho<EOS>(P, rho, psi_c);
            if (in1)
#pragma unroll
                for (int k = 0; k < 9; ++k) L.a1[k][l1] = fb[k];
            if (wall_row) {
                if (y == 1) { L.rv1[0][lx] = rx; L.rv1[1][lx] = ry; }
                if (y == P.ny - 2) { L.rv1[2][lx] = rx; L.rv1[3][lx] = ry; }
            }
        }
        L.q1x[tid] = qx;
        L.q1y[tid] = qy;
    }
    __syncthreads();
    if (in1) L.c1[l1] = act ? dpsi1 * adj_xi(P, L.q1x, L.q1y, W2, tid, y, p01) : 0.0;
    __syncthreads();
    if (!second || !act) return;

    // ---- the second step on the tile ----
    const int l = (ly + 1) * W1 + lx + 1;
    const double* cc = L.sp2 + l;
    double sx, sy, nu[9], fb[9], pb, qx, qy, rx, ry;
    cohesion_sum(cc[-W1 - 1], cc[-W1], cc[-W1 + 1], cc[-1], cc[1], cc[W1 - 1], cc[W1], cc[W1 + 1],
                 sx, sy);
    push_gather_lds(P, L.a1, L.c1, W1, l, y, nu);
    collide_adj(P, f, rho, psi_c, sx, sy, Ax, Ay, nu, fb, pb, qx, qy, rx, ry);
    const unsigned i = (unsigned)y * P.pitch + x;
#pragma unroll
    for (int k = 0; k < 9; ++k) (A.a_out + k * P.plane)[i] = fb[k];
    A.q_out[i] = qx;
    (A.q_out + P.plane)[i] = qy;
    A.p0_out[i] = pb;
    A.dpsi_out[i] = dpsi_drho<EOS>(P, rho, psi_c);
    if (wall_row) {
        if (y == 1) { A.rv_out[x] = rx; A.rv_out[P.pitch + x] = ry; }
        if (y == P.ny - 2) { A.rv_out[2 * P.pitch + x] = rx; A.rv_out[3 * P.pitch + x] = ry; }
        adj_gw_node(P, A.rv_in, A.gwgrad, x, y);
        adj_gw_sum(P, L.rv1[0], W2, lx + 1, lx + 2, lx + 3, A.gwgrad, x, y);
    }
}

}  // namespace lbm
