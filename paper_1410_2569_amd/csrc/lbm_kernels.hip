// lbm_kernels.hip -- gfx950 kernels of the wetting pseudopotential LB step and its observables.
//
// Step schedules (both call the same per-node arithmetic of lbm_device.h):
//   fused     one kernel per time step. A workgroup owns a TX x TY tile; every thread pulls the
//             9 populations of its node (Eq. 5 with bounce-back), forms rho and psi, and the
//             psi of the one-node tile halo is recomputed from the (L2-resident) populations of
//             the neighbouring tiles. psi lives only in LDS, so HBM sees 72 B read + 72 B
//             written per lattice update.
//   two-pass  psi pass (pull, rho, psi -> psi array with mirrored ghost rows), then the step
//             kernel stages the psi tile plus halo in LDS: 72 + 8 B and 72 + 8 + 72 B per update.
//   two-step  two time steps per launch with the intermediate state in LDS (step2_tile).
//   multi-step four time steps per launch on lattices too small to fill the GPU (steps_tile).
//   marching  three time steps per launch on large lattices: strips of columns march through
//             registers (march_strip).
// With the wet-node wall scheme the boundary nodes also write their force (16 B) to the solid row,
// which the next pull reads back; that traffic is confined to two rows of the lattice.
#include <algorithm>
#include <map>
#include <type_traits>
#include <utility>
#include <vector>

#include "lbm_device.h"
#include "lbm_internal.h"
#include "lbm_march.h"
#include "lbm_obs.h"
#include "lbm_steps.h"
#include "lbm_wave.h"

namespace lbm {

// ------------------------------------------------------------------------------------------------
// Time step
// ------------------------------------------------------------------------------------------------
// GEO, EOS: the geometry and equation-of-state variants compiled in, chosen at launch.
template <int TX, int TY, bool FUSED, int GEO, int EOS>
__global__ __launch_bounds__(TX* TY) void k_step(KParams P, const double* __restrict__ gin,
                                                 double* __restrict__ gout,
                                                 const double* __restrict__ psi_g,
                                                 const double* __restrict__ gw) {
    __shared__ double sp[(TY + 2) * (TX + 2)];
    const int ntx = (P.nx + TX - 1) / TX;
    const int nty = (P.y_hi - P.y_lo + TY) / TY;
    const int tile = xcd_tile(blockIdx.x, ntx * nty);
    step_tile<TX, TY, FUSED, GEO, EOS>(P, gin, gout, psi_g, gw, (tile % ntx) * TX,
                                       P.y_lo + (tile / ntx) * TY, sp);
}

// Overlapped tiles: one 64-lane wave spans TXI = 62 interior columns plus the halo column on each
// side, and the workgroup has TYI interior rows plus a halo row above and below. Every thread
// pulls exactly one node and evaluates its psi (one memory round trip per tile, all loads
// coalesced rows); the interior threads then collide and store.
template <int TYI, int GEO, int EOS>
__global__ __launch_bounds__(64 * (TYI + 2)) void k_step_ov(KParams P,
                                                            const double* __restrict__ gin,
                                                            double* __restrict__ gout,
                                                            const double* __restrict__ gw) {
    constexpr int TXI = 62, LW = 64;
    __shared__ double sp[(TYI + 2) * LW];
    const int ntx = (P.nx + TXI - 1) / TXI;
    const int nty = (P.y_hi - P.y_lo + TYI) / TYI;
    const int tile = xcd_tile(blockIdx.x, ntx * nty);
    const int x0 = (tile % ntx) * TXI;
    const int y0 = P.y_lo + (tile / ntx) * TYI;
    const int l = threadIdx.x & 63, r = threadIdx.x >> 6;
    const int gx = x0 - 1 + l, gy = y0 - 1 + r;
    const bool interior = l >= 1 && l <= TXI && r >= 1 && r <= TYI && gx < P.nx && gy <= P.y_hi;

    int sx, sy;
    const bool has = slot_source(P, gx, gy, sx, sy);
    double f[9];
    double rho = 1.0, psi_c = 0.0;
    if (has) {
        pull9<GEO>(P, gin, sx, sy, f);
        rho = sum9(f);
        psi_c = psi_of_rho<EOS>(P, rho);
    }
    sp[r * LW + l] = psi_c;
    __syncthreads();
    if (!interior) return;

    const double* c = sp + r * LW + l;
    double sxx, syy;
    cohesion_sum(c[-LW - 1], c[-LW], c[-LW + 1], c[-1], c[1], c[LW - 1], c[LW], c[LW + 1], sxx,
                 syy);
    double Ax = 0.0, Ay = 0.0;
    if (P.walls && (gy == 1 || gy == P.ny - 2)) adhesion_sum(P, gw, gx, gy, Ax, Ay);
    store_wall_force<GEO>(P, gout, (long long)gy * P.pitch + gx, P.plane, P.pitch, gy, rho, psi_c,
                          sxx, syy, Ax, Ay);
    collide(P, f, rho, psi_c, sxx, syy, Ax, Ay);
    const unsigned i = (unsigned)gy * P.pitch + gx;
#pragma unroll
    for (int a = 0; a < 9; ++a) (gout + a * P.plane)[i] = f[a];
}

// Two steps per launch over TX x TY output tiles (step2_tile) with NTH threads; MID: the state
// after the first step is written to gmid as well.
template <int TX, int TY, int GEO, int EOS, bool MID, int NTH = step2_threads(TX, TY, GEO)>
__global__ __launch_bounds__(NTH, NTH == step2_threads(TX, TY, GEO)
                                      ? step2_waves(TX, TY, GEO)
                                      : (NTH / 64 + 3) / 4) void k_step2(
    KParams P, const double* __restrict__ gin, double* __restrict__ gout,
    const double* __restrict__ gw, double* __restrict__ gmid) {
    __shared__ Step2Lds<TX, TY, GEO> lds;
    const int ntx = (P.nx + TX - 1) / TX;
    const int nty = (P.y_hi - P.y_lo + TY) / TY;
    const int tile = xcd_tile(blockIdx.x, ntx * nty);
    step2_tile_any<TX, TY, GEO, EOS, MID, false, NTH>(P, gin, gout, gw, (tile % ntx) * TX,
                                                      P.y_lo + (tile / ntx) * TY, lds, gmid);
}

// kTileSteps steps per launch over TX x TY output tiles (steps_tile).
template <int TX, int TY, int GEO, int EOS, bool MID>
__global__ __launch_bounds__(steps_threads(kTileSteps, TX, TY)) void k_steps(
    KParams P, const double* __restrict__ gin, double* __restrict__ gout,
    const double* __restrict__ gw, double* __restrict__ mid, long long mstride) {
    __shared__ StepsLds<kTileSteps, TX, TY, GEO> lds;
    const int ntx = (P.nx + TX - 1) / TX;
    const int nty = (P.y_hi - P.y_lo + TY) / TY;
    const int t = xcd_tile(blockIdx.x, ntx * nty);
    steps_tile<kTileSteps, TX, TY, GEO, EOS, MID>(P, gin, gout, gw, (t % ntx) * TX,
                                                  P.y_lo + (t / ntx) * TY, lds, mid, mstride);
}

// kMarchSteps steps per launch: every wave marches one strip through one segment of h rows
// (march_strip). Two waves per SIMD, 256 registers each: three levels take 237 to 241 of them, and
// with the wet-node wall or Eq. (15) compiled in up to all, of which most such variants spill 4 to 14
// (8 to 35 in the ensembles' kernel, which holds two viscosities' code). The spills lie in the set-up
// and in the rows beside a wall or seam; no plain row touches scratch memory, and the variants run
// alike: 2048 x 1024 30.6 us per step with bounce-back and Carnahan-Starling, 30.5 with both.
template <int GEO, int EOS, int VISC>
__global__ __launch_bounds__(64 * kMarchWaves, 2) void k_march(
    KParams P, const double* __restrict__ gin, double* __restrict__ gout,
    const double* __restrict__ gw, int nstrips, int nseg, int h) {
    const int n = nstrips * nseg;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = xcd_tile(blockIdx.x, gridDim.x) * kMarchWaves + wave;
    if (w >= n) return;
    const int seg = w / nstrips, strip = w - seg * nstrips;
    const int y0 = P.y_lo + seg * h;
    const int y1 = y0 + h - 1 < P.y_hi ? y0 + h - 1 : P.y_hi;
    march_strip<kMarchSteps, GEO, EOS, VISC, DppLane>(P, gin, gout, gw,
                                                      strip * march_cols(kMarchSteps), y0, y1,
                                                      threadIdx.x & 63);
}

// psi pass of the two-pass schedule; also writes the mirrored ghost rows.
__global__ __launch_bounds__(256) void k_psi(KParams P, const double* __restrict__ gin,
                                             double* __restrict__ psi_g) {
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = P.y_lo + blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= P.nx || y > P.y_hi) return;
    psi_node(P, gin, psi_g, nullptr, x, y);
}

// ------------------------------------------------------------------------------------------------
// State set-up and read-out
// ------------------------------------------------------------------------------------------------

// Inverse of streaming + bounce-back: writes g so that the first pull yields f_a = t_a rho0.
// Every post-collision slot of a fluid node is the source of exactly one pulled population.
__global__ __launch_bounds__(256) void k_init(KParams P, const double* __restrict__ rho0,
                                              double* __restrict__ g) {
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = P.y_lo + blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= P.nx || y > P.y_hi) return;
    if (is_solid_node(P, x, y)) return;
    const double r = rho0[(long long)y * P.pitch + x];
    const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    const int op[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
    const unsigned lk = P.mask ? P.links[(unsigned)y * P.pitch + x] : 0u;
    for (int a = 0; a < 9; ++a) {
        const double t = a == 0 ? 4.0 / 9.0 : (a < 5 ? 1.0 / 9.0 : 1.0 / 36.0);
        int sx = wrapx(x - ex[a], P.nx);
        int sy = y - ey[a];
        bool solid = false;
        if (P.mask) { solid = (lk >> a) & 1u; sy = wrapx(sy, P.ny); }
        else if (P.walls) solid = (sy == 0 || sy == P.ny - 1);
        else sy = wrapx(sy, P.ny);
        if (solid) g[op[a] * P.plane + (long long)y * P.pitch + x] = t * r;
        else g[a * P.plane + (long long)sy * P.pitch + sx] = t * r;
    }
}

// Read-out of every node of the lattice, dense and complete (0 on solid nodes), so that the copy to
// the host is all that follows: pre-collision populations f^n [9][ny][nx], or with RHO the density
// [ny][nx].
template <bool RHO>
__global__ __launch_bounds__(256) void k_read(KParams P, const double* __restrict__ gin,
                                              double* __restrict__ out) {
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= P.nx || y >= P.ny) return;
    double f[9] = {};
    if (y >= P.y_lo && y <= P.y_hi && !is_solid_node(P, x, y)) pull9_any(P, gin, x, y, f);
    const long long pl = (long long)P.nx * P.ny, i = (long long)y * P.nx + x;
    if (RHO) {
        out[i] = sum9(f);
    } else {
#pragma unroll
        for (int a = 0; a < 9; ++a) out[a * pl + i] = f[a];
    }
}

// Copy of `planes` planes of ny rows of nx doubles between two layouts in device memory: rows
// src_pitch doubles apart (planes src_plane apart) to rows dst_pitch apart (planes dst_plane
// apart). Host data enter and leave the library densely packed through it, so that every copy
// between host and device memory is one contiguous transfer.
__global__ __launch_bounds__(256) void k_repack(const double* __restrict__ src, long long src_plane,
                                                int src_pitch, double* __restrict__ dst,
                                                long long dst_plane, int dst_pitch, int nx,
                                                int ny, int planes) {
    const long long per = (long long)ny * nx, n = per * planes;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (long long)gridDim.x * 256) {
        const long long a = i / per, r = i - a * per;
        const long long y = r / nx, x = r - y * nx;
        dst[a * dst_plane + y * dst_pitch + x] = src[a * src_plane + y * src_pitch + x];
    }
}

// ------------------------------------------------------------------------------------------------
// Observables (obs_tile, obs_final_block)
// ------------------------------------------------------------------------------------------------
template <bool PRE, int ROWS>
__global__ __launch_bounds__(256) void k_obs(KParams P, const double* __restrict__ gin,
                                             const double* __restrict__ gw, ObsArgs A,
                                             double* __restrict__ part) {
    __shared__ ObsLds<ROWS> lds;
    obs_tile<PRE, ROWS>(P, gin, gw, A, blockIdx.x, blockIdx.y, gridDim.x, part, lds);
}

__global__ __launch_bounds__(256) void k_obs_final(const double* __restrict__ part, int nblk,
                                                   double* __restrict__ out) {
    __shared__ double sh[O_NQ][256];
    obs_final_block(part, nblk, sh, out);
}

// Contact line of one lattice (contact_line_block).
__global__ __launch_bounds__(256) void k_contact_line(KParams P, const double* __restrict__ gin,
                                                      int row, double mid,
                                                      double* __restrict__ out) {
    contact_line_block(P, gin, row, mid, out);
}

// Zero fill of n 8-byte words (grid-stride). The library clears its buffers with this kernel
// rather than a runtime memset, so the clear is ordered like every other kernel of the stream.
__global__ __launch_bounds__(256) void k_zero(unsigned long long* __restrict__ p, size_t n) {
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

// ------------------------------------------------------------------------------------------------
// Host-side launchers
// ------------------------------------------------------------------------------------------------
static dim3 node_grid(const KParams& P) {
    return dim3((P.nx + 63) / 64, (P.y_hi - P.y_lo + 4) / 4);
}

// Calls f(geo, eos) with the geometry and equation of state of P as compile-time constants.
template <class F>
static hipError_t dispatch(const KParams& P, F&& f) {
    auto with_eos = [&](auto geo) {
        if (P.eos == 0) return f(geo, std::integral_constant<int, EOS_CS>{});
        return f(geo, std::integral_constant<int, EOS_PW>{});
    };
    if (P.mask) return with_eos(std::integral_constant<int, GEO_MASK>{});
    if (P.wet) return with_eos(std::integral_constant<int, GEO_WET>{});
    return with_eos(std::integral_constant<int, GEO_ROWS>{});
}

template <int TX, int TY, bool FUSED>
static hipError_t launch_step_t(const KParams& P, const double* gin, double* gout,
                                const double* psi, const double* gw, hipStream_t s) {
    const int ntx = (P.nx + TX - 1) / TX;
    const int nty = (P.y_hi - P.y_lo + TY) / TY;
    return dispatch(P, [&](auto geo, auto eos) {
        hipLaunchKernelGGL((k_step<TX, TY, FUSED, decltype(geo)::value, decltype(eos)::value>),
                           dim3(ntx * nty), dim3(TX * TY), 0, s, P, gin, gout, psi, gw);
        return hipGetLastError();
    });
}

// The overlapped tiles have no solid-mask variant (the API rejects those schedules for a
// mask).
template <int TYI>
static hipError_t launch_step_ov(const KParams& P, const double* gin, double* gout,
                                 const double* gw, hipStream_t s) {
    const int ntx = (P.nx + 61) / 62;
    const int nty = (P.y_hi - P.y_lo + TYI) / TYI;
    return dispatch(P, [&](auto geo, auto eos) {
        if constexpr (decltype(geo)::value == GEO_MASK) {
            return hipErrorInvalidValue;
        } else {
            hipLaunchKernelGGL((k_step_ov<TYI, decltype(geo)::value, decltype(eos)::value>),
                               dim3(ntx * nty), dim3(64 * (TYI + 2)), 0, s, P, gin, gout, gw);
            return hipGetLastError();
        }
    });
}

template <int TX, int TY, bool WIDE = false>
static hipError_t launch_step2_t(const KParams& P, const double* gin, double* gout,
                                 const double* gw, double* gmid, hipStream_t s) {
    const int ntx = (P.nx + TX - 1) / TX;
    const int nty = (P.y_hi - P.y_lo + TY) / TY;
    return dispatch(P, [&](auto geo, auto eos) {
        constexpr int G = decltype(geo)::value;
        constexpr int E = decltype(eos)::value;
        constexpr int NT = WIDE ? step2_wide_threads(TX, TY) : step2_threads(TX, TY, G);
        if (!gmid) {
            hipLaunchKernelGGL((k_step2<TX, TY, G, E, false, NT>), dim3(ntx * nty), dim3(NT), 0,
                               s, P, gin, gout, gw, (double*)nullptr);
            return hipGetLastError();
        }
        if constexpr (G == GEO_ROWS) {
            hipLaunchKernelGGL((k_step2<TX, TY, G, E, true, NT>), dim3(ntx * nty), dim3(NT), 0,
                               s, P, gin, gout, gw, gmid);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;  // intermediate states: bounce-back or periodic rows only
        }
    });
}

// Two steps in one launch; tile2 selects the output tile: 0 64x8, 1 64x4, 2 128x4, 3 64x16,
// 4 32x8, 5 32x4 (the narrow tiles for lattices too small to fill the chip with the others), 6
// 64x4 and 7 32x4 with wide workgroups (step2_wide_threads).
// gmid (optional): receives the state after the first step.
hipError_t launch_step2(const KParams& P, int tile2, const double* gin, double* gout,
                        const double* gw, hipStream_t s, double* gmid) {
    switch (tile2) {
        case 1: return launch_step2_t<64, 4>(P, gin, gout, gw, gmid, s);
        case 2: return launch_step2_t<128, 4>(P, gin, gout, gw, gmid, s);
        case 3: return launch_step2_t<64, 16>(P, gin, gout, gw, gmid, s);
        case 4: return launch_step2_t<32, 8>(P, gin, gout, gw, gmid, s);
        case 5: return launch_step2_t<32, 4>(P, gin, gout, gw, gmid, s);
        case 6: return launch_step2_t<64, 4, true>(P, gin, gout, gw, gmid, s);
        case 7: return launch_step2_t<32, 4, true>(P, gin, gout, gw, gmid, s);
        default: return launch_step2_t<64, 8>(P, gin, gout, gw, gmid, s);
    }
}

// Multi-step tiles. The smallest tile that gives every compute unit at most one workgroup (the
// halo's work per workgroup is then the least), or 16 x 8 up to two per compute unit: 300 x 150 (361
// tiles) 3.47 -> 3.18 us per step, 340 x 140 (396) 3.87 -> 3.23. Beyond, the halo's work tells:
// 384 x 192 (576 tiles) 3.82 -> 4.39.
int steps_tile_of(int nx, int rows) {
    auto tiles = [&](int tx, int ty) { return (long long)((nx + tx - 1) / tx) * ((rows + ty - 1) / ty); };
    if (tiles(8, 4) <= 256) return 0;
    if (tiles(8, 8) <= 256) return 1;
    return tiles(16, 8) <= 512 ? 2 : -1;
}

template <int TX, int TY>
static hipError_t launch_steps_t(const KParams& P, const double* gin, double* gout,
                                 const double* gw, double* mid, long long mstride, hipStream_t s) {
    const int ntx = (P.nx + TX - 1) / TX;
    const int nty = (P.y_hi - P.y_lo + TY) / TY;
    return dispatch(P, [&](auto geo, auto eos) {
        constexpr int G = decltype(geo)::value, E = decltype(eos)::value;
        constexpr int NT = steps_threads(kTileSteps, TX, TY);
        if (!mid) {
            hipLaunchKernelGGL((k_steps<TX, TY, G, E, false>), dim3(ntx * nty), dim3(NT), 0, s, P,
                               gin, gout, gw, mid, mstride);
            return hipGetLastError();
        }
        if constexpr (G == GEO_ROWS) {
            hipLaunchKernelGGL((k_steps<TX, TY, G, E, true>), dim3(ntx * nty), dim3(NT), 0, s, P,
                               gin, gout, gw, mid, mstride);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    });
}

hipError_t launch_steps(const KParams& P, int tile, const double* gin, double* gout,
                        const double* gw, hipStream_t s, double* mid, long long mstride) {
    switch (tile) {
        case 0: return launch_steps_t<8, 4>(P, gin, gout, gw, mid, mstride, s);
        case 1: return launch_steps_t<8, 8>(P, gin, gout, gw, mid, mstride, s);
        default: return launch_steps_t<16, 8>(P, gin, gout, gw, mid, mstride, s);
    }
}

// Marching strips: the split into segments, and the launch.
static int strips_of(const MarchShape& m) {
    constexpr int C = march_cols(kMarchSteps);
    return (m.nx + C - 1) / C;
}

// Rows per segment for `count` lattices, or 0 where the two-step tiles are faster. The split is
// chosen by the time of one launch: every wave walks its segment's rows and the 4T-2 halo rows, the
// SIMDs run one wave each or two at a time (a third round is a second pass over the chip, so the
// number of waves should fall just below a multiple of 2048), and a launch costs about 7 us before
// its first full row. Measured per row: 1.75 us with one wave per SIMD, 2.9 us for two
// (2048 x 1024: 26 segments of 40 rows, 988 waves, 96 us per launch; 52 of 20, 1976 waves, 92 us;
// 32 of 32, 1216 waves, 116 us). The two-step tiles make 49 updates per ns on a full chip. The
// line lies near a million nodes: 1024 x 512 takes 10.9 us per step with tiles and 12.4 marching (14.3
// with periodic rows), 1400 x 700 17.4-18.3 and 17.2-17.5 (18.2), 1500 x 1001 25.3 and 22.5-24.1,
// 2048 x 1024 40.3 and 30.6, 4096 x 4096 312 and 212. With the wet-node wall and Eq. (15) the same
// within 5%: 13.1, 17.3, 22.7, 30.5, 211.
int march_rows(const MarchShape* m, int count) {
    constexpr int H = 2 * kMarchSteps - 1;
    double nodes = 0.0;
    // Strips by the rows that they are cut into: the loop below weighs up to a thousand splits, and
    // an ensemble has few different heights (3,000 lattices of six: 11 ms one by one, 0.4 so).
    std::map<int, long long> by_rows;
    for (int i = 0; i < count; ++i) {
        if (m[i].rows < 16 || m[i].nx > (1 << 28)) return 0;
        by_rows[m[i].rows] += strips_of(m[i]);
        nodes += (double)m[i].nx * m[i].rows;
    }
    const std::vector<std::pair<int, long long>> strips(by_rows.begin(), by_rows.end());
    const int rmax = strips.back().first;
    int best = 0;
    double best_us = 0.0;
    auto waves_at = [&](int h) {
        long long n = 0;
        for (const auto& [rows, k] : strips) n += k * ((rows + h - 1) / h);
        return n;
    };
    for (int h = std::min(rmax, 1024); h >= 8; --h) {
        const long long n = waves_at(h);
        const double us = n <= kSimds ? 7.0 + 1.75 * (h + 2 * H)
                                      : 7.0 + 2.9 * (h + 2 * H) * ((n + 2 * kSimds - 1) / (2 * kSimds));
        if (!best || us < best_us) {
            best = h;
            best_us = us;
        }
    }
    return best_us < 0.95 * (3.0 * nodes / 49000.0) ? best : 0;
}

void march_segments(const MarchShape& m, int inst, int y_lo, int h, std::vector<MarchSeg>* out) {
    constexpr int C = march_cols(kMarchSteps);
    const int nseg = (m.rows + h - 1) / h, hh = (m.rows + nseg - 1) / nseg;
    for (int s = 0; s * hh < m.rows; ++s)
        for (int x0 = 0; x0 < m.nx; x0 += C)
            out->push_back({inst, x0, y_lo + s * hh, y_lo + std::min(m.rows, (s + 1) * hh) - 1});
}

hipError_t launch_march(const KParams& P, int h, const double* gin, double* gout, const double* gw,
                        hipStream_t s) {
    const int rows = P.y_hi - P.y_lo + 1;
    const int nstrips = strips_of({P.nx, rows}), nseg = (rows + h - 1) / h;
    const int blocks = (nstrips * nseg + kMarchWaves - 1) / kMarchWaves;
    return dispatch(P, [&](auto geo, auto eos) {
        constexpr int G = decltype(geo)::value, E = decltype(eos)::value;
        if constexpr (G == GEO_MASK) {
            return hipErrorInvalidValue;
        } else {
            if (P.visc_const)
                hipLaunchKernelGGL((k_march<G, E, 1>), dim3(blocks), dim3(64 * kMarchWaves), 0, s,
                                   P, gin, gout, gw, nstrips, nseg, h);
            else
                hipLaunchKernelGGL((k_march<G, E, 2>), dim3(blocks), dim3(64 * kMarchWaves), 0, s,
                                   P, gin, gout, gw, nstrips, nseg, h);
            return hipGetLastError();
        }
    });
}

// Fused tile shapes: 0-3 halo-recompute tiles TX x TY; 4-7 overlapped tiles 62 x TYI.
static const int kTiles[8][3] = {{64, 4, 0}, {64, 8, 0}, {64, 16, 0}, {128, 4, 0},
                                 {62, 4, 1}, {62, 6, 1}, {62, 8, 1}, {62, 14, 1}};

int n_tiles() { return 8; }

void tile_shape(int tile, int* tx, int* ty) {
    if (tile < 0 || tile >= 8) tile = 0;
    *tx = kTiles[tile][0];
    *ty = kTiles[tile][1];
}

hipError_t launch_step(const KParams& P, int schedule, int tile, const double* gin, double* gout,
                       double* psi, const double* gw, hipStream_t s) {
    if (schedule == 1) {
        hipLaunchKernelGGL(k_psi, node_grid(P), dim3(256), 0, s, P, gin, psi);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_step_t<64, 4, false>(P, gin, gout, psi, gw, s);
    }
    switch (tile) {
        case 1: return launch_step_t<64, 8, true>(P, gin, gout, psi, gw, s);
        case 2: return launch_step_t<64, 16, true>(P, gin, gout, psi, gw, s);
        case 3: return launch_step_t<128, 4, true>(P, gin, gout, psi, gw, s);
        case 4: return launch_step_ov<4>(P, gin, gout, gw, s);
        case 5: return launch_step_ov<6>(P, gin, gout, gw, s);
        case 6: return launch_step_ov<8>(P, gin, gout, gw, s);
        case 7: return launch_step_ov<14>(P, gin, gout, gw, s);
        default: return launch_step_t<64, 4, true>(P, gin, gout, psi, gw, s);
    }
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s) {
    if (bytes % 8 || ((uintptr_t)p) % 8) return hipErrorInvalidValue;
    const size_t n = bytes / 8;
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_zero, dim3(blocks), dim3(256), 0, s, (unsigned long long*)p, n);
    return hipGetLastError();
}

// SplitMix64 (S. Vigna's public-domain mixer): add the golden-ratio increment, then two
// xor-shift-multiply rounds and a final xor-shift, all modulo 2^64.
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Initial density of liquid droplets in their vapour on every node of the lattice (pitched
// rows): the largest of the droplets' tanh profiles, times 1 + jitter (2u - 1) with u the
// node's uniform of the seeded counter stream; 0 on solid rows.
__global__ __launch_bounds__(256) void k_droplets(KParams P, DropletArgs D, double* __restrict__ rho) {
#pragma clang fp contract(off)
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= P.nx || y >= P.ny) return;
    double v = 0.0;
    if (y >= P.y_lo && y <= P.y_hi) {
        v = -INFINITY;
        for (int k = 0; k < D.count; ++k) {
            const double dx = x - D.x0[k], dy = y - D.y0[k];
            const double d = sqrt(dx * dx + dy * dy);
            const double rk = D.mid - D.half * tanh(2.0 * (d - D.r[k]) / D.width);
            v = fmax(v, rk);
        }
        if (D.jitter != 0.0) {
            const unsigned long long z =
                splitmix64(D.base + (unsigned long long)y * (unsigned long long)P.nx + x);
            const double u = (double)(z >> 11) * 0x1.0p-53;
            v = v * (1.0 + D.jitter * (2.0 * u - 1.0));
        }
    }
    rho[(long long)y * P.pitch + x] = v;
}

hipError_t launch_droplets(const KParams& P, const DropletArgs& D, double* rho, hipStream_t s) {
    hipLaunchKernelGGL(k_droplets, dim3((P.nx + 63) / 64, (P.ny + 3) / 4), dim3(256), 0, s, P, D,
                       rho);
    return hipGetLastError();
}

// The device's FP64 square root and division, element-wise: sq = sqrt(a), qt = a / b. Operands of
// magnitudes well inside the range of doubles, as the step's are, take its root() and quot() (recip()
// is quot() of 1, operation by operation). The rest take the compiler's, which know zeros,
// infinities and subnormal numbers.
__global__ __launch_bounds__(256) void k_fp64_probe(const double* __restrict__ a,
                                                    const double* __restrict__ b,
                                                    double* __restrict__ sq,
                                                    double* __restrict__ qt, long long n) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    auto inside = [](double v) { return fabs(v) >= 0x1p-500 && fabs(v) <= 0x1p500; };
    sq[i] = inside(a[i]) ? root(a[i]) : sqrt(a[i]);
    qt[i] = inside(a[i]) && inside(b[i]) ? quot(a[i], b[i]) : a[i] / b[i];
}

hipError_t launch_fp64_probe(const double* a, const double* b, double* sq, double* quot,
                             long long n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fp64_probe, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, b,
                       sq, quot, n);
    return hipGetLastError();
}

hipError_t launch_init(const KParams& P, const double* rho0, double* g, hipStream_t s) {
    hipLaunchKernelGGL(k_init, node_grid(P), dim3(256), 0, s, P, rho0, g);
    return hipGetLastError();
}

hipError_t launch_read(const KParams& P, const double* gin, double* out, bool rho, hipStream_t s) {
    const dim3 g((P.nx + 63) / 64, (P.ny + 3) / 4);
    if (rho) hipLaunchKernelGGL(k_read<true>, g, dim3(256), 0, s, P, gin, out);
    else hipLaunchKernelGGL(k_read<false>, g, dim3(256), 0, s, P, gin, out);
    return hipGetLastError();
}

hipError_t launch_repack(const double* src, long long src_plane, int src_pitch, double* dst,
                         long long dst_plane, int dst_pitch, int nx, int ny, int planes,
                         hipStream_t s) {
    const long long n = (long long)planes * ny * nx;
    if (n <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<long long>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_repack, dim3(blocks), dim3(256), 0, s, src, src_plane, src_pitch, dst,
                       dst_plane, dst_pitch, nx, ny, planes);
    return hipGetLastError();
}

hipError_t launch_contact_line(const KParams& P, const double* gin, int row, double mid,
                               double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_contact_line, dim3(1), dim3(256), 0, s, P, gin, row, mid, out);
    return hipGetLastError();
}

int obs_blocks(const KParams& P) { return obs_rows(P); }

hipError_t launch_obs(const KParams& P, const double* gin, const double* gw, const ObsArgs& A,
                      double* part, double* out, hipStream_t s, bool pre) {
    auto go = [&](auto rows) {
        constexpr int R = decltype(rows)::value;
        const dim3 g((P.nx + 63) / 64, (P.y_hi - P.y_lo + R) / R);
        if (pre) hipLaunchKernelGGL((k_obs<true, R>), g, dim3(256), 0, s, P, gin, gw, A, part);
        else hipLaunchKernelGGL((k_obs<false, R>), g, dim3(256), 0, s, P, gin, gw, A, part);
        return hipGetLastError();
    };
    hipError_t e = obs_rows(P) < 512 ? go(std::integral_constant<int, kObsRowsSmall>{})
                                     : go(std::integral_constant<int, kObsRows>{});
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_obs_final, dim3(1), dim3(256), 0, s, part, obs_rows(P), out);
    return hipGetLastError();
}

}  // namespace lbm
