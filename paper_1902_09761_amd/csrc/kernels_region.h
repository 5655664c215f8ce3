// Regions of the fused 2D preconditioner kernels (gfx950): the inner operators in split form, sweeps over
// register-resident rows of regions one wave wide, and the walk of a thread's rows over the periodic mesh.
#pragma once

#include "kernels_common.h"

namespace apfc {

__device__ __forceinline__ int wrapi(int g, int n) {
    g %= n;
    return g < 0 ? g + n : g;
}

// The operators of the inner solves in split form.  With P = [1 4 1], Q = [-1 2 -1] = 6 delta - P and
// E = [-1 0 1], the bilinear element stencils are M = (h/6)^2 P(x)P,
// K = (1/6)(Q(x)P + P(x)Q) = (delta(x)P + P(x)delta) - P(x)P/3 and T_j = (h/6)(k0 E(x)P + k1 P(x)E).
// At a node with rows A, B, C (y - 1, y, y + 1), x passes p = P u and e = E u of those rows and centre
// values uA, uB, uC:
//   (cM M + cK K) u = a (pA + pC) + b pB + c (uA + uC) + d uB,
//   a = cM (h/6)^2 - cK/3,  b = 4 a + cK,  c = cK,  d = 4 cK   (M alone: a = (h/6)^2, b = 4 a, c = d = 0),
//   T_j u = (h/6) (k0 (eA + 4 eB + eC) + k1 (pC - pA)).

// Sweep of a region one wave wide (64 columns, the thread's lane is its column) with the thread's NP rows
// u[] in registers: the x neighbours come by lane shifts (0 beyond the region's outer columns, whose
// values only reach the halo), the rows above and below the thread's block from the neighbouring waves
// through edge[w][0] and edge[w][1] (first and last row of the block of wave w; 0 above the first block and
// below the last, as the pad rows of the LDS region).  One barrier, after the edge rows are stored.
// f(i, ...) is called as by split_sweep, in row order, and may overwrite u[i] (read by then).
template <typename T, int NP, int NW, bool WE, typename F>
__device__ __forceinline__ void reg_sweep(cx<T> (&u)[NP], cx<T> (*edge)[2][kTX], int w, F&& f) {
    const int lane = (int)threadIdx.x & (kTX - 1);
    edge[w][0][lane] = u[0];
    edge[w][1][lane] = u[NP - 1];
    __syncthreads();
    const cx<T> zero{T(0), T(0)};
    const cx<T> above = w > 0 ? edge[w - 1][1][lane] : zero;
    const cx<T> below = w + 1 < NW ? edge[w + 1][0][lane] : zero;
    auto xpass = [&](cx<T> c, cx<T>& p, cx<T>& e) {
        const cx<T> l = lane_shift<kDppWaveShr1>(c), r = lane_shift<kDppWaveShl1>(c);
        p = T(4) * c + (l + r);
        e = WE ? r - l : zero;
    };
    cx<T> uA = above, uB = u[0], pA, pB, eA, eB;
    xpass(uA, pA, eA);
    xpass(uB, pB, eB);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const cx<T> uC = i + 1 < NP ? u[i + 1] : below;
        cx<T> pC, eC;
        xpass(uC, pC, eC);
        f(i, pA, pB, pC, uA, uB, uC, eA, eB, eC);
        uA = uB;
        uB = uC;
        pA = pB;
        pB = pC;
        eA = eB;
        eB = eC;
    }
}

// The same walk with the x pass left to the caller: make(l, c, r) forms a row's pass from a node and its x
// neighbours, f(i, A, B, C, uB) gets the passes of rows y - 1, y, y + 1 and the node's value.
template <typename T, int NP, int NW, typename MAKE, typename F>
__device__ __forceinline__ void row_sweep(cx<T> (&u)[NP], cx<T> (*edge)[2][kTX], int w, MAKE&& make, F&& f) {
    const int lane = (int)threadIdx.x & (kTX - 1);
    edge[w][0][lane] = u[0];
    edge[w][1][lane] = u[NP - 1];
    __syncthreads();
    const cx<T> zero{T(0), T(0)};
    const cx<T> above = w > 0 ? edge[w - 1][1][lane] : zero;
    const cx<T> below = w + 1 < NW ? edge[w + 1][0][lane] : zero;
    auto pass = [&](cx<T> c) { return make(lane_shift<kDppWaveShr1>(c), c, lane_shift<kDppWaveShl1>(c)); };
    auto A = pass(above);
    auto B = pass(u[0]);
    cx<T> uB = u[0];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const cx<T> uC = i + 1 < NP ? u[i + 1] : below;
        auto C = pass(uC);
        f(i, A, B, C, uB);
        A = B;
        B = C;
        uB = uC;
    }
}

// stencil() for a walk over rows: x passes m = mass u, k = (stiffness u) h and e = derivative u of a row, and M u,
// K u, T u from three of them, with the contractions the compiler makes of stencil(), where a node's nine
// values are in one block.
template <typename T>
struct RowStencil {
    struct Row {
        cx<T> m, k, e;
    };
    T m0, m1, ih, cM, cK;
    __device__ explicit RowStencil(const Sys& s) {
        const T h = T(s.h);
        m0 = h * T(1.0 / 6.0);
        m1 = h * T(4.0 / 6.0);
        ih = T(1) / h;
        cM = T(s.isq_dt);
        cK = T(s.sq_kap);
    }
    __device__ __forceinline__ Row row(cx<T> l, cx<T> c, cx<T> r) const {
        return {m0 * (l + r) + m1 * c, (c + c) - (l + r), T(0.5) * (r - l)};
    }
    __device__ __forceinline__ cx<T> M(const Row& A, const Row& B, const Row& C) const {
        return m0 * (A.m + C.m) + m1 * B.m;
    }
    __device__ __forceinline__ cx<T> K(const Row& A, const Row& B, const Row& C) const {
        const cx<T> kc = ih * C.k;
        const cx<T> ks{mad(ih, A.k.x, kc.x), mad(ih, A.k.y, kc.y)};
        return (m0 * ks + m1 * (ih * B.k)) + ih * ((B.m + B.m) - (A.m + C.m));
    }
    __device__ __forceinline__ cx<T> Tj(const Row& A, const Row& B, const Row& C, T k0, T k1) const {
        const cx<T> x = k0 * (m0 * (A.e + C.e) + m1 * B.e), y = T(0.5) * (C.m - A.m);
        return cx<T>{T(2) * mad(k1, y.x, x.x), T(2) * mad(k1, y.y, x.y)};
    }
    __device__ __forceinline__ cx<T> L(const Row& A, const Row& B, const Row& C) const {
        return cM * M(A, B, C) + cK * K(A, B, C);
    }
};

struct SplitCoef {
    double a, b, c, d;
};
__host__ __device__ inline SplitCoef split_coef(double h, double cM, double cK) {
    const double m = (h / 6.0) * (h / 6.0), a = cM * m - cK / 3.0;
    return {a, 4.0 * a + cK, cK, 4.0 * cK};
}

// Global node of the thread's region rows: x wrapped once per thread, rows walked with a running
// periodic row index (no division per row).
struct RegionRows {
    long long base, gx;
    int gy, nx, ny;
    __device__ __forceinline__ long long at() const { return base + (long long)gy * nx + gx; }
    __device__ __forceinline__ void next() { gy = gy + 1 == ny ? 0 : gy + 1; }
};

// The region of workgroup blockIdx.x of system blockIdx.y, 64 x (NP NW) nodes with `halo` layers around an interior
// tile, tiles row by row; init: false past the system's last one.
template <int NP, int NW>
struct Region {
    RegionRows rows0;
    int x0, y0, ix, r0, IX, IY, nx, ny;
    __device__ __forceinline__ bool init(const Sys& s, int halo) {
        nx = s.nx;
        ny = s.ny;
        IX = kTX - 2 * halo;
        IY = NP * NW - 2 * halo;
        const int nrx = (nx + IX - 1) / IX, nry = (ny + IY - 1) / IY, b = (int)blockIdx.x;
        if (b >= nrx * nry) return false;
        x0 = (b % nrx) * IX;
        y0 = (b / nrx) * IY;
        const int lane = (int)threadIdx.x & 63;
        r0 = ((int)threadIdx.x >> 6) * NP - halo;
        ix = lane - halo;
        rows0 = RegionRows{s.off, (long long)wrapi(x0 + ix, nx), wrapi(y0 + r0, ny), nx, ny};
        return true;
    }
    __device__ __forceinline__ bool owned(int i) const {
        const int iy = r0 + i;
        return ix >= 0 && ix < IX && x0 + ix < nx && iy >= 0 && iy < IY && y0 + iy < ny;
    }
};

}  // namespace apfc
