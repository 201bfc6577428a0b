// lbm_obs.h -- observables of one lattice, reduced block by block in a fixed order: per-block
// partials (wave-level shuffles, then LDS across waves), then one block over the partials. No
// floating-point atomics, so results are bitwise reproducible, and the same for a lattice alone and
// in an ensemble.
#pragma once
#include "lbm_device.h"

namespace lbm {

// LDS of obs_tile: density and psi of 64 x 8 nodes and one ring, partials of 4 waves.
constexpr int kObsRows = 8;
struct ObsLds {
    double rho[(kObsRows + 2) * 66], psi[(kObsRows + 2) * 66];
    double red[kObsRows / 4][4][O_NQ];
};

// Observables of the 64 x 8 nodes at (64 bx, y_lo + 8 by), by 256 threads, two nodes each: density
// and psi of the nodes and the ring around them are formed in LDS from the pulled populations (no
// field goes through memory), then every wave reduces its 64 nodes of each row. Writes the O_NQ
// partials of each half of 64 x 4 nodes, part[(2 by + half) * nbx + bx], where it holds fluid rows.
// Waves without an interface crossing or a node that is not finite (most) skip those sums, whose
// every term is 0. What bounds it: one read of the populations; the ring's pulls come from L2.
template <bool PRE>
__device__ __forceinline__ void obs_tile(const KParams& P, const double* __restrict__ gin,
                                         const double* __restrict__ gw, const ObsArgs& A, int bx,
                                         int by, int nbx, double* __restrict__ part, ObsLds& L) {
    constexpr int LW = 66, NR = kObsRows / 4, NRING = 2 * LW + 2 * kObsRows;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int x0 = bx * 64, y0 = P.y_lo + by * kObsRows, x = x0 + lane;
    double f[NR][9];
    bool act[NR];
    // density and psi at lattice slot (gx, gy); 0 where the slot holds none
    auto slot = [&](int gx, int gy, double g[9], double& rho) {
        int sx, sy;
        rho = 0.0;
        if (!slot_source(P, gx, gy, sx, sy)) return 0.0;
        node_populations<PRE>(P, gin, sx, sy, g);
        rho = sum9(g);
        return psi_of_rho(P, rho);
    };
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int ly = 4 * r + wv, y = y0 + ly;
        act[r] = x < P.nx && y <= P.y_hi && !is_solid_node(P, x, y);
        const int l = (ly + 1) * LW + lane + 1;
        L.psi[l] = slot(x, y, f[r], L.rho[l]);
    }
    for (int h = threadIdx.x; h < NRING; h += 256) {
        int lx, ly;
        if (h < LW) { lx = h; ly = 0; }
        else if (h < 2 * LW) { lx = h - LW; ly = kObsRows + 1; }
        else if (h < 2 * LW + kObsRows) { lx = 0; ly = h - 2 * LW + 1; }
        else { lx = LW - 1; ly = h - 2 * LW - kObsRows + 1; }
        double g[9];
        L.psi[ly * LW + lx] = slot(x0 - 1 + lx, y0 - 1 + ly, g, L.rho[ly * LW + lx]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int y = y0 + 4 * r + wv;
        double v[O_NQ];
        for (int q = 0; q < O_NQ; ++q) v[q] = op_identity(q);
        if (act[r]) {
            const int l = (4 * r + wv + 1) * LW + lane + 1;
            const double* c = L.psi + l;
            const double w[9] = {c[-LW - 1], c[-LW], c[-LW + 1], c[-1],    c[0],
                                 c[1],       c[LW - 1], c[LW],   c[LW + 1]};
            obs_values(P, f[r], L.rho[l], w, gw, A, x, y, L.rho[l + 1], L.rho[l + LW], v);
        }
        const bool fit = __any(v[O_N] != 0.0), bad = __any(v[O_BAD] != 0.0);
#pragma unroll
        for (int q = 0; q < O_NQ; ++q) {
            double s = v[q];
            if (q < O_BAD || (q == O_BAD && bad) || (q > O_BAD && fit))
                for (int off = 32; off > 0; off >>= 1)
                    s = op_combine(q, s, __shfl_xor(s, off, 64));
            if (lane == 0) L.red[r][wv][q] = s;
        }
    }
    __syncthreads();
    const int r = threadIdx.x >> 4, q = threadIdx.x & 15;
    if (r < NR && q < O_NQ && y0 + 4 * r <= P.y_hi) {
        const double s = op_combine(q, op_combine(q, L.red[r][0][q], L.red[r][1][q]),
                                    op_combine(q, L.red[r][2][q], L.red[r][3][q]));
        part[(long long)((NR * by + r) * nbx + bx) * O_NQ + q] = s;
    }
}

// The partial rows that obs_tile writes for a lattice: 64 x 4 nodes each.
__host__ __device__ inline int obs_rows(const KParams& P) {
    return (P.nx + 63) / 64 * ((P.y_hi - P.y_lo + 4) / 4);
}

// One block of 256 threads: for every quantity, thread t combines partials t, t+256, ... in
// order, then a fixed tree; all quantities advance together (one pass over the partial rows).
__device__ __forceinline__ void obs_final_block(const double* __restrict__ part, int nblk,
                                                double (*sh)[256], double* __restrict__ out) {
    double s[O_NQ];
#pragma unroll
    for (int q = 0; q < O_NQ; ++q) s[q] = op_identity(q);
    for (int b = threadIdx.x; b < nblk; b += 256) {
        const double* r = part + (long long)b * O_NQ;
#pragma unroll
        for (int q = 0; q < O_NQ; ++q) s[q] = op_combine(q, s[q], r[q]);
    }
#pragma unroll
    for (int q = 0; q < O_NQ; ++q) sh[q][threadIdx.x] = s[q];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
#pragma unroll
            for (int q = 0; q < O_NQ; ++q)
                sh[q][threadIdx.x] = op_combine(q, sh[q][threadIdx.x], sh[q][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if ((int)threadIdx.x < O_NQ) out[threadIdx.x] = sh[threadIdx.x][0];
}

}  // namespace lbm
