// lbm_obs.h -- observables of one lattice, reduced block by block in a fixed order: per-block
// partials (wave-level shuffles, then LDS across waves), then one block over the partials. No
// floating-point atomics, so results are bitwise reproducible, and the same for a lattice alone and
// in an ensemble.
#pragma once
#include "lbm_device.h"

namespace lbm {

// LDS of obs_tile: density and psi of 64 x ROWS nodes and one ring, partials of 4 waves.
template <int ROWS>
struct ObsLds {
    double rho[(ROWS + 2) * 66], psi[(ROWS + 2) * 66];
    double red[ROWS / 4][4][O_NQ];
};
// Rows of a block: 8, or 4 on lattices with fewer than 256 blocks of 8, whose compute units would
// wait for one block's longer chain (100 x 50: 45.4 us per call with 8, 40.7 with 4; two passes
// over the lattice took 44.1).
constexpr int kObsRows = 8, kObsRowsSmall = 4;

// Observables of the 64 x ROWS nodes at (64 bx, y_lo + ROWS by), by 256 threads: density
// and psi of the nodes and the ring around them are formed in LDS from the pulled populations (no
// field goes through memory), then every wave reduces its 64 nodes of each row. Writes the O_NQ
// partials of each 64 x 4 nodes, part[(ROWS / 4 by + r) * nbx + bx], where they hold fluid rows.
// Waves without an interface crossing or a node that is not finite (most) skip those sums, whose
// every term is 0. What bounds it: one read of the populations; the ring's pulls come from L2.
// 1024 x 512, a call on held populations: 67.8 us with two passes and their fields, 57.5 so.
template <bool PRE, int ROWS>
__device__ __forceinline__ void obs_tile(const KParams& P, const double* __restrict__ gin,
                                         const double* __restrict__ gw, const ObsArgs& A, int bx,
                                         int by, int nbx, double* __restrict__ part, ObsLds<ROWS>& L) {
    constexpr int LW = 66, NR = ROWS / 4, NRING = 2 * LW + 2 * ROWS;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int x0 = bx * 64, y0 = P.y_lo + by * ROWS, x = x0 + lane;
    // every pull is issued before the first psi: two nodes and, for some threads, a slot of the ring
    double f[NR][9], g[9];
    bool act[NR], has[NR], hasg = false;
    auto pull = [&](int gx, int gy, double p[9]) {
        int sx, sy;
        if (!slot_source(P, gx, gy, sx, sy)) return false;
        node_populations<PRE>(P, gin, sx, sy, p);
        return true;
    };
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int y = y0 + 4 * r + wv;
        act[r] = x < P.nx && y <= P.y_hi && !is_solid_node(P, x, y);
        has[r] = pull(x, y, f[r]);
    }
    static_assert(NRING <= 256, "at most one slot of the ring per thread");
    const int h = threadIdx.x;
    int lx, ly;
    if (h < LW) { lx = h; ly = 0; }
    else if (h < 2 * LW) { lx = h - LW; ly = ROWS + 1; }
    else if (h < 2 * LW + ROWS) { lx = 0; ly = h - 2 * LW + 1; }
    else { lx = LW - 1; ly = h - 2 * LW - ROWS + 1; }
    if (h < NRING) hasg = pull(x0 - 1 + lx, y0 - 1 + ly, g);
    // density and psi into slot l; 0 where the slot holds none
    auto put = [&](bool v, const double p[9], int l) {
        const double rho = v ? sum9(p) : 0.0;
        L.rho[l] = rho;
        L.psi[l] = v ? psi_of_rho(P, rho) : 0.0;
    };
#pragma unroll
    for (int r = 0; r < NR; ++r) put(has[r], f[r], (4 * r + wv + 1) * LW + lane + 1);
    if (h < NRING) put(hasg, g, ly * LW + lx);
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
