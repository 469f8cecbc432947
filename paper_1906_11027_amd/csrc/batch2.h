// batch2.h -- an item of a batched sweep, and the kernel that advances the items
// two steps per launch with the node arithmetic of the including unit.
#pragma once
#include "tile2.h"

namespace sclbm {

template <typename T>
struct BatchItem {
    const T* a;          // state buffer 0
    T* b;                // state buffer 1
    int nx, ny;
    int order;           // 4, 6, 8, 10
    T gc0, omega, guo;
};

constexpr int kBRMAX = 3;   // largest stencil radius

// Two steps per launch: the two-step tile of the single-grid kernel
// (tile2.h) per work entry, with the item's stencil order (a uniform switch)
// and LDS sized for the largest radius.  Work entries of one item are listed
// in strip order; the XCD swizzle gives each XCD a contiguous range of them,
// so tiles that share halo lines run on the same XCD (same L2).
template <typename T, class Node, int TX, int TY, int NT>
__global__ void __launch_bounds__(NT)
k_d2q9_batch2(const BatchItem<T>* __restrict__ items, const int2* __restrict__ work, int parity,
              StepArgs<T> common)
{
    using LD = Tile2Lds<kBRMAX, TX, TY>;
    __shared__ T psi1[LD::P1N];
    __shared__ T psi2[LD::P2N];
    __shared__ T s1[9 * LD::C1N];
    const int2 wk = work[xcd_swizzle(blockIdx.x, gridDim.x)];
    const BatchItem<T> it = items[wk.x];
    StepArgs<T> a = common;
    a.fin = parity ? it.b : it.a;
    a.fout = parity ? (T*)it.a : it.b;
    a.nx = it.nx;
    a.ny = it.ny;
    a.nz = 1;
    a.n = (int64_t)it.nx * it.ny;
    a.gc0 = it.gc0;
    a.omega = it.omega;
    a.guo = it.guo;
    const int tiles_x = (it.nx + TX - 1) / TX;
    const int x0 = (wk.y % tiles_x) * TX, y0 = (wk.y / tiles_x) * TY;
    switch (it.order) {   // uniform across the block
    case 4: d2q9_tile2_body<T, Node, 4, TX, TY, NT>(a, x0, y0, psi1, psi2, s1); break;
    case 6: d2q9_tile2_body<T, Node, 6, TX, TY, NT>(a, x0, y0, psi1, psi2, s1); break;
    case 8: d2q9_tile2_body<T, Node, 8, TX, TY, NT>(a, x0, y0, psi1, psi2, s1); break;
    default: d2q9_tile2_body<T, Node, 10, TX, TY, NT>(a, x0, y0, psi1, psi2, s1); break;
    }
}

// The shape of 32 x 8 tiles, in the single grids' arithmetic
// (kernels_batch_grid.hip).
template <typename T>
hipError_t launch_batch_grid(const BatchItem<T>* items, const int2* work, int nwork, int parity, const StepArgs<T>& common,
                             hipStream_t s);

}  // namespace sclbm
