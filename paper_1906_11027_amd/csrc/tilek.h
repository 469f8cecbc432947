// tilek.h -- K time steps per launch with one node per thread, for grids so
// small that the launches and the latency of each phase are the cost: shared
// by the D2Q9 (Guo) kernels and the any-lattice 2D kernels.
#pragma once
#include "kernels.h"

namespace sclbm {

// The interaction force at LDS node c of rows of LW nodes (Sec. 2, Eq. (1)).
template <typename T, int ORDER>
__device__ __forceinline__ void tile_force_at(const T* c, int LW, T gc0, T& Fx, T& Fy)
{
    T sx, sy;
    force_sums<T, ORDER>([&](int ex, int ey) { return c[ey * LW + ex]; }, sx, sy);
    const T pref = -gc0 * c[0];
    Fx = pref * sx;
    Fy = pref * sy;
}

// Regions of a TX x TY tile advanced K steps: with S = R + M (force radius
// plus lattice reach) step k collides the tile + (K - k) S and needs psi on R
// more nodes around that, so the first step pulls the tile + (K - 1) S + R.
template <class Mod, int ORDER, int TX, int TY, int K>
struct TileK {
    static constexpr int R = Stencil<2, ORDER>::R, S = R + Mod::M;
    static constexpr int HP = (K - 1) * S + R, PW = TX + 2 * HP, PN = PW * (TY + 2 * HP);
    static constexpr int HC = (K - 1) * S, CW = TX + 2 * HC, CN = K > 1 ? CW * (TY + 2 * HC) : 0;
    static constexpr int NT = (PN + 63) / 64 * 64;   // one node per thread
};

// What bounds it: on a grid of 64^2 to 200 x 100 nodes a step is a chain of
// launch, load latency, barriers and one node's arithmetic per wave, with most
// of the chip idle.  So every node of the pulled region has its own thread
// (all loads in flight at once, one pass per phase), the tiles are small (more
// compute units, fewer waves on each), and K steps share one launch and one
// trip to memory.  A thread keeps its node through all steps: the node's wall
// flag and coordinates stay in registers, and each step takes two barriers
// (psi complete; post-collision values complete).  The values pulled for a step
// are in registers before the first barrier, so one copy s1 serves all steps.
// us per step, against the two-step tiles with several nodes per thread or the
// one-step tiles whose halo ring is pulled one node at a time: D2Q9 E4 FP64 64^2
// 1.85 / 2.5 (four steps), D2Q13 E6 FP64 60^2 2.94 / 4.9 (two), D2Q25 E8 FP64 with
// walls 200 x 100 5.3 / 7.9 (two), 1001 x 777 E8 FP32 30.6 / 33.8 (one).
template <typename T, class Mod, int ORDER, bool WALLS, int TX, int TY, int K, int NT>
__global__ void __launch_bounds__(NT)
k_tile_steps(StepArgs<T> a, int nbx)
{
    using W = TileK<Mod, ORDER, TX, TY, K>;
    using L = typename Mod::L;
    constexpr int Q = Mod::Q, M = Mod::M, R = W::R, S = W::S, PW = W::PW;
    __shared__ T psi[W::PN];
    __shared__ T s1[K > 1 ? Q * W::CN : 1];

    const int nx = a.nx, ny = a.ny;
    const int64_t n = a.n;
    const uint32_t TS = sizeof(T), rowb = (uint32_t)nx * TS;
    const int tile = xcd_swizzle(blockIdx.x, gridDim.x);
    const int x0 = (tile % nbx) * TX, y0 = (tile / nbx) * TY;
    const int i = threadIdx.x;
    const int py = i / PW, px = i - py * PW;
    const int tx = px - W::HP, ty = py - W::HP;   // from the tile's corner
    // the node lies on the tile + h
    auto within = [&](int h) { return tx >= -h && tx < TX + h && ty >= -h && ty < TY + h; };
    const int ci = (ty + W::HC) * W::CW + tx + W::HC;   // its place in s1, where it has one

    T g[Q];
    bool wall = false;
    if (i < W::PN) {
        uint32_t xo[2 * M + 1], yo[2 * M + 1];
#pragma unroll
        for (int k = 0; k <= 2 * M; ++k) {
            xo[k] = (uint32_t)wrap_near(x0 + tx - M + k, nx) * TS;
            yo[k] = (uint32_t)wrap_near(y0 + ty - M + k, ny) * rowb;
        }
#pragma unroll
        for (int b = 0; b < Q; ++b) g[b] = ld_off(a.fin + b * n, yo[M - L::cy[b]] + xo[M - L::cx[b]]);
        if constexpr (WALLS) wall = a.solid[(yo[M] + xo[M]) / TS];
    }
#pragma unroll
    for (int k = 1; k <= K; ++k) {
        const int hc = (K - k) * S;
        T dr = T(0);
        if (within(hc + R) && i < W::PN) {
            if (k > 1) {
#pragma unroll
                for (int b = 0; b < Q; ++b) g[b] = s1[b * W::CN + ci - L::cy[b] * W::CW - L::cx[b]];
            }
            dr = Mod::sum(g);
            psi[i] = wall ? a.psi_w : psi_of(a.rho_ref + dr, a);
        }
        __syncthreads();
        if (within(hc)) {
            if (WALLS && wall) {
                T r[Q];
#pragma unroll
                for (int b = 0; b < Q; ++b) r[b] = g[Mod::opposite(b)];
#pragma unroll
                for (int b = 0; b < Q; ++b) g[b] = r[b];
            } else {
                T Fx, Fy;
                tile_force_at<T, ORDER>(psi + i, PW, a.gc0, Fx, Fy);
                Mod::collide(g, dr, Fx, Fy, a);
            }
            if (k < K) {
#pragma unroll
                for (int b = 0; b < Q; ++b) s1[b * W::CN + ci] = g[b];
            } else if (x0 + tx < nx && y0 + ty < ny) {
                const uint32_t own = (uint32_t)(y0 + ty) * rowb + (uint32_t)(x0 + tx) * TS;
#pragma unroll
                for (int b = 0; b < Q; ++b) st_off(a.fout + b * n, own, g[b]);
            }
        }
        if (k < K) __syncthreads();
    }
}

template <typename T, class Mod, int ORDER, bool WALLS, int TX, int TY, int K>
static hipError_t launch_tile_steps(const StepArgs<T>& a, hipStream_t s)
{
    using W = TileK<Mod, ORDER, TX, TY, K>;
    constexpr int fit = tile_steps_fit(W::R, Mod::M, Mod::Q, sizeof(T), TX, TY, K);
    if constexpr (fit != K) {
        return launch_tile_steps<T, Mod, ORDER, WALLS, TX, TY, fit>(a, s);
    } else {
        const int nbx = (a.nx + TX - 1) / TX, nby = (a.ny + TY - 1) / TY;
        hipLaunchKernelGGL((k_tile_steps<T, Mod, ORDER, WALLS, TX, TY, K, W::NT>), dim3(nbx * nby), dim3(W::NT), 0, s,
                           a, nbx);
        return hipGetLastError();
    }
}

}  // namespace sclbm
