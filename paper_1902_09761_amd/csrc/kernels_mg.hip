// Geometric multigrid V-cycle for the diffusion operator L = M/sqrt(dt) + sqrt(kappa) K of the block
// preconditioner (Eq. (12)), the multigrid variant of its inner solves (Sec. III), on the structured mesh:
// levels of twice the mesh size, coarse operators by rediscretisation (the same stencil with the
// level's h, equal to the Galerkin product for the Q1 interpolation), symmetric Chebyshev-Jacobi
// smoothing (the level's Sys::cb[1] table: the upper part of the spectrum of D^{-1} L), restriction by
// the transpose of the Q1 interpolation, and a coarsest level solved in LDS by Chebyshev iterations over
// its whole spectrum.  One cycle from a zero initial guess:
//     x = S(b);  r = b - L x;  x += P V(P^T r);  r = b - L x;  x += S(r).
#include "kernels_region.h"

namespace apfc {

// (L u) at the node of n, u in the level's half vector
template <int DIM, typename T>
__device__ __forceinline__ cx<T> apply_L(const Sys& s, const Nbr<DIM>& n, const cx<T>* u) {
    cx<T> Mu, Ku, Tu;
    stencil<DIM, true, false, T>([&](int a, int b, int c) { return ld<T>(u, s.off + nb_index<DIM>(n, a, b, c)); },
                                 T(s.h), T(0), T(0), T(0), Mu, Ku, Tu);
    return T(s.isq_dt) * Mu + T(s.sq_kap) * Ku;
}

// Start of a smoothing pass.  ADD = false (from a zero guess): r = b, d = c0 b, x = d.
// ADD = true (a correction from the residual r): d = c0 r, x += d.
template <int DIM, int TY, typename T, bool ADD>
__global__ __launch_bounds__(kBlock) void k_mg_start(const Sys* sys, const Tile* tiles, const int* mask, const cx<T>* b,
                                                    cx<T>* r, cx<T>* d, cx<T>* xv) {
    TILE_PROLOGUE();
    const T c0 = T(sys[tile.sys].cb[1][0][0]);
    FOR_ROWS(TY) {
        const long long i = s.off + ((long long)pz * s.ny + y) * s.nx + x;
        if constexpr (ADD) {
            const cx<T> dv = c0 * ld<T>(r, i);
            d[i] = dv;
            xv[i] = ld<T>(xv, i) + dv;
        } else {
            const cx<T> bv = ld<T>(b, i);
            const cx<T> dv = c0 * bv;
            r[i] = bv;
            d[i] = dv;
            xv[i] = dv;
        }
    }
}

// Chebyshev iteration j >= 1 on L: r -= L d_{j-1}; d_j = c1 d_{j-1} + c2 r; x += d_j (LAST: r and d_j are
// not stored)
template <int DIM, int TY, typename T, bool LAST>
__global__ __launch_bounds__(kBlock) void k_mg_iter(const Sys* sys, const Tile* tiles, const int* mask, int j,
                                                   const cx<T>* din, cx<T>* dout, cx<T>* r, cx<T>* xv) {
    TILE_PROLOGUE();
    const T c1 = T(sys[tile.sys].cb[1][j][0]), c2 = T(sys[tile.sys].cb[1][j][1]);
    FOR_ROWS(TY) {
        Nbr<DIM> n;
        make_nbr<DIM>(s, x, y, pz, n);
        const long long i = s.off + nb_index<DIM>(n, 1, 1, 1);
        const cx<T> rv = ld<T>(r, i) - apply_L<DIM, T>(s, n, din);
        const cx<T> dv = c1 * ld<T>(din, i) + c2 * rv;
        xv[i] = ld<T>(xv, i) + dv;
        if constexpr (!LAST) {
            r[i] = rv;
            dout[i] = dv;
        }
    }
}

// r = b - L x
template <int DIM, int TY, typename T>
__global__ __launch_bounds__(kBlock) void k_mg_residual(const Sys* sys, const Tile* tiles, const int* mask,
                                                       const cx<T>* b, const cx<T>* xv, cx<T>* r) {
    TILE_PROLOGUE();
    FOR_ROWS(TY) {
        Nbr<DIM> n;
        make_nbr<DIM>(s, x, y, pz, n);
        const long long i = s.off + nb_index<DIM>(n, 1, 1, 1);
        r[i] = ld<T>(b, i) - apply_L<DIM, T>(s, n, xv);
    }
}

// Restriction b_c = P^T r_f on the coarse level's tiles: coarse node I gathers the fine nodes 2I + a,
// a in {-1, 0, 1}^dim (periodic), with weight prod_d (a_d == 0 ? 1 : 1/2).  fsys: the fine level's table
// (the same system index).
template <int DIM, int TY, typename T>
__global__ __launch_bounds__(kBlock) void k_mg_restrict(const Sys* sys, const Tile* tiles, const int* mask,
                                                       const Sys* fsys, const cx<T>* rf, cx<T>* bc) {
    TILE_PROLOGUE();
    const Sys f = fsys[tile.sys];
    FOR_ROWS(TY) {
        const int fx = 2 * x, fy = 2 * y, fz = 2 * pz;
        const int xs[3] = {fx == 0 ? f.nx - 1 : fx - 1, fx, fx + 1 == f.nx ? 0 : fx + 1};
        const int ys[3] = {fy == 0 ? f.ny - 1 : fy - 1, fy, fy + 1 == f.ny ? 0 : fy + 1};
        const int zs[3] = {DIM == 3 ? (fz == 0 ? f.nz - 1 : fz - 1) : 0, fz, DIM == 3 ? (fz + 1 == f.nz ? 0 : fz + 1) : 0};
        const T w[3] = {T(0.5), T(1), T(0.5)};
        cx<T> acc{T(0), T(0)};
#pragma unroll
        for (int c = (DIM == 3 ? 0 : 1); c < (DIM == 3 ? 3 : 2); ++c)
#pragma unroll
            for (int bb = 0; bb < 3; ++bb)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const T wt = w[a] * w[bb] * (DIM == 3 ? w[c] : T(1));
                    const long long fi = f.off + ((long long)zs[c] * f.ny + ys[bb]) * f.nx + xs[a];
                    acc = acc + wt * ld<T>(rf, fi);
                }
        bc[s.off + ((long long)pz * s.ny + y) * s.nx + x] = acc;
    }
}

// Prolongation x_f += P x_c on the fine level's tiles: per direction an even fine index 2i takes coarse
// node i, an odd one 2i + 1 the mean of coarse nodes i and i + 1 (periodic); tensor product.
template <int DIM, int TY, typename T>
__global__ __launch_bounds__(kBlock) void k_mg_prolong(const Sys* sys, const Tile* tiles, const int* mask,
                                                      const Sys* csys, const cx<T>* xc, cx<T>* xf) {
    TILE_PROLOGUE();
    const Sys c = csys[tile.sys];
    FOR_ROWS(TY) {
        int ix[2], iy[2], iz[2];
        T wx[2], wy[2], wz[2];
        auto par = [](int f, int nc, int (&i)[2], T (&w)[2]) {
            i[0] = f >> 1;
            if (f & 1) {
                i[1] = i[0] + 1 == nc ? 0 : i[0] + 1;
                w[0] = w[1] = T(0.5);
            } else {
                i[1] = i[0];
                w[0] = T(1);
                w[1] = T(0);
            }
        };
        par(x, c.nx, ix, wx);
        par(y, c.ny, iy, wy);
        if constexpr (DIM == 3) par(pz, c.nz, iz, wz);
        else { iz[0] = iz[1] = 0; wz[0] = T(1); wz[1] = T(0); }
        cx<T> acc{T(0), T(0)};
#pragma unroll
        for (int cz = 0; cz < 2; ++cz)
#pragma unroll
            for (int cy = 0; cy < 2; ++cy)
#pragma unroll
                for (int cxi = 0; cxi < 2; ++cxi) {
                    const T wt = wx[cxi] * wy[cy] * wz[cz];
                    if (wt != T(0))
                        acc = acc + wt * ld<T>(xc, c.off + ((long long)iz[cz] * c.ny + iy[cy]) * c.nx + ix[cxi]);
                }
        const long long i = s.off + ((long long)pz * s.ny + y) * s.nx + x;
        xf[i] = ld<T>(xf, i) + acc;
    }
}

// Coarsest level: x = Chebyshev^its(b) from zero over the whole spectrum (the level's cb[1] table), one
// workgroup per system with the level's correction d in LDS (at most kMgCoarseMax nodes), r and x of the
// thread's nodes in registers.
constexpr int kMgThreads = 1024;
constexpr int kMgPerThread = kMgCoarseMax / kMgThreads;

template <int DIM, typename T>
__global__ __launch_bounds__(kMgThreads) void k_mg_coarse(const Sys* sys, const int* mask, int its, const cx<T>* b,
                                                        cx<T>* xout) {
    __shared__ cx<T> dl[kMgCoarseMax];
    const int si = blockIdx.x;
    if (mask && !mask[si]) return;
    const Sys s = sys[si];
    const int N = (int)s.N;
    const double(*cb)[2] = sys[si].cb[1];
    const T cM = T(s.isq_dt), cK = T(s.sq_kap);
    cx<T> r[kMgPerThread], xv[kMgPerThread], dv[kMgPerThread];
    const T c0 = T(cb[0][0]);
#pragma unroll
    for (int q = 0; q < kMgPerThread; ++q) {
        const int i = (int)threadIdx.x + q * kMgThreads;
        if (i < N) {
            r[q] = ld<T>(b, s.off + i);
            dv[q] = c0 * r[q];
            xv[q] = dv[q];
        }
    }
    for (int k = 1; k < its; ++k) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kMgPerThread; ++q) {
            const int i = (int)threadIdx.x + q * kMgThreads;
            if (i < N) dl[i] = dv[q];
        }
        __syncthreads();
        const T c1 = T(cb[k][0]), c2 = T(cb[k][1]);
#pragma unroll
        for (int q = 0; q < kMgPerThread; ++q) {
            const int i = (int)threadIdx.x + q * kMgThreads;
            if (i >= N) continue;
            const int ix = i % s.nx, iy = (i / s.nx) % s.ny, iz = DIM == 3 ? i / (s.nx * s.ny) : 0;
            const int xs[3] = {ix == 0 ? s.nx - 1 : ix - 1, ix, ix + 1 == s.nx ? 0 : ix + 1};
            const int ys[3] = {iy == 0 ? s.ny - 1 : iy - 1, iy, iy + 1 == s.ny ? 0 : iy + 1};
            const int zs[3] = {DIM == 3 ? (iz == 0 ? s.nz - 1 : iz - 1) : 0, iz, DIM == 3 ? (iz + 1 == s.nz ? 0 : iz + 1) : 0};
            cx<T> Mu, Ku, Tu;
            stencil<DIM, true, false, T>([&](int a, int bb, int c) { return dl[(zs[c] * s.ny + ys[bb]) * s.nx + xs[a]]; },
                                         T(s.h), T(0), T(0), T(0), Mu, Ku, Tu);
            r[q] = r[q] - (cM * Mu + cK * Ku);
            dv[q] = c1 * dv[q] + c2 * r[q];
            xv[q] = xv[q] + dv[q];
        }
    }
#pragma unroll
    for (int q = 0; q < kMgPerThread; ++q) {
        const int i = (int)threadIdx.x + q * kMgThreads;
        if (i < N) xout[s.off + i] = xv[q];
    }
}

// ------------------------------------------------------------------------------------------
// Fused 2D V-cycle, up to kMgFusedNu smoothing iterations: a level above 64 x 64 nodes takes one launch down
// and one up on register-resident regions of 64 x 32 nodes (row_sweep), the levels below one launch for all of
// them (k_mg_tail).  Per node the arithmetic and its rounding are those of the kernels above.  Latency bounds
// the cycle (a level of 128 x 112 x 3 is 45 regions): 2 levels + 1 launches of 6 to 15 us and one of 35 us
// instead of 7 launches per level of ~4.5 us each and the coarsest level's 29 us; 512 x 448 x 3, dt = 10: a step
// of 55 FGMRES iterations 25.9 -> 12.7 ms.
// ------------------------------------------------------------------------------------------
constexpr int kMgFusedNu = 4, kMgNP = 4, kMgNW = 8, kMgRegY = kMgNP * kMgNW, kMgRegThreads = 64 * kMgNW;

using MgRegion = Region<kMgNP, kMgNW>;

template <typename T>
struct Raw {
    cx<T> l, c, r;
};
// sum of the 3 x 3 fine nodes with weights (1/2, 1, 1/2) x (1/2, 1, 1/2), in the order of k_mg_restrict
template <typename T>
__device__ __forceinline__ cx<T> mg_restrict(const Raw<T>& A, const Raw<T>& B, const Raw<T>& C) {
    const T q = T(0.25), h = T(0.5);
    cx<T> a = q * A.l;
    a = a + h * A.c;
    a = a + q * A.r;
    a = a + h * B.l;
    a = a + B.c;
    a = a + h * B.r;
    a = a + q * C.l;
    a = a + h * C.c;
    return a + q * C.r;
}
// (P x_c) at fine node (gx, gy), ld(i, j) = node (i, j) of the coarse level of nx x ny nodes, in the order of
// k_mg_prolong
template <typename T, typename F>
__device__ __forceinline__ cx<T> mg_interp(int gx, int gy, int nx, int ny, F&& ld) {
    const int i0 = gx >> 1, j0 = gy >> 1, i1 = i0 + 1 == nx ? 0 : i0 + 1, j1 = j0 + 1 == ny ? 0 : j0 + 1;
    const bool ox = gx & 1, oy = gy & 1;
    const T w = (ox ? T(0.5) : T(1)) * (oy ? T(0.5) : T(1));
    cx<T> a = w * ld(i0, j0);
    if (ox) a = a + w * ld(i1, j0);
    if (oy) a = a + w * ld(i0, j1);
    if (ox && oy) a = a + w * ld(i1, j1);
    return a;
}

// Down: x = S(b) (to xs, read by the way up), r = b - L x, b_c = P^T r (to bc, the coarse level's half vector).
// RHS 0: b = src; 1: b = v - kappa G src (step 2); 2: b = M src (step 3); formed b is stored to bout.
template <typename T, int RHS>
__global__ __launch_bounds__(kMgRegThreads) void k_mg_down2d(const Sys* sys, const Sys* csys, const int* mask,
                                                            const cx<T>* v, const cx<T>* src, cx<T>* bout, cx<T>* xs,
                                                            cx<T>* bc, int nu, int halo) {
    __shared__ cx<T> edges[2][kMgNW][2][kTX];
    const int si = blockIdx.y, wv = (int)threadIdx.x >> 6;
    if (mask && !mask[si]) return;
    const Sys& s = sys[si];
    MgRegion reg;
    if (!reg.init(s, halo)) return;
    using Row = typename RowStencil<T>::Row;
    const RowStencil<T> st(s);
    auto make = [&](cx<T> l, cx<T> c, cx<T> r) { return st.row(l, c, r); };
    int e = 0;
    cx<T> B[kMgNP], R[kMgNP], D[kMgNP], X[kMgNP];
    {
        RegionRows g = reg.rows0;
#pragma unroll
        for (int i = 0; i < kMgNP; ++i, g.next()) D[i] = src[g.at()];
    }
    if constexpr (RHS == 0) {
#pragma unroll
        for (int i = 0; i < kMgNP; ++i) B[i] = D[i];
    } else {
        if constexpr (RHS == 1) {
            RegionRows g = reg.rows0;
#pragma unroll
            for (int i = 0; i < kMgNP; ++i, g.next()) B[i] = v[g.at()];
        }
        const T k0 = T(s.kv[0]), k1 = T(s.kv[1]), kap = T(s.kappa);
        row_sweep<T, kMgNP, kMgNW>(D, edges[e], wv, make, [&](int i, const Row& a, const Row& b, const Row& c, cx<T>) {
            if constexpr (RHS == 1)
                B[i] = B[i] - kap * gop(st.K(a, b, c), st.Tj(a, b, c, k0, k1));
            else
                B[i] = st.M(a, b, c);
        });
        e ^= 1;
        RegionRows g = reg.rows0;
#pragma unroll
        for (int i = 0; i < kMgNP; ++i, g.next())
            if (reg.owned(i)) bout[g.at()] = B[i];
    }
    const double(*cb)[2] = s.cb[1];
    const T c0 = T(cb[0][0]);
#pragma unroll
    for (int i = 0; i < kMgNP; ++i) {
        R[i] = B[i];
        D[i] = c0 * B[i];
        X[i] = D[i];
    }
    for (int j = 1; j < nu; ++j) {
        const T c1 = T(cb[j][0]), c2 = T(cb[j][1]);
        row_sweep<T, kMgNP, kMgNW>(D, edges[e], wv, make,
                                   [&](int i, const Row& a, const Row& b, const Row& c, cx<T> dB) {
                                       R[i] = R[i] - st.L(a, b, c);
                                       D[i] = c1 * dB + c2 * R[i];
                                       X[i] = X[i] + D[i];
                                   });
        e ^= 1;
    }
    {
        RegionRows g = reg.rows0;
#pragma unroll
        for (int i = 0; i < kMgNP; ++i, g.next())
            if (reg.owned(i)) xs[g.at()] = X[i];
    }
    row_sweep<T, kMgNP, kMgNW>(X, edges[e], wv, make, [&](int i, const Row& a, const Row& b, const Row& c, cx<T>) {
        R[i] = B[i] - st.L(a, b, c);
    });
    e ^= 1;
    const Sys& cs = csys[si];
    row_sweep<T, kMgNP, kMgNW>(
        R, edges[e], wv, [](cx<T> l, cx<T> c, cx<T> r) { return Raw<T>{l, c, r}; },
        [&](int i, const Raw<T>& a, const Raw<T>& b, const Raw<T>& c, cx<T>) {
            const int gx = reg.x0 + reg.ix, gy = reg.y0 + reg.r0 + i;
            if (reg.owned(i) && !(gx & 1) && !(gy & 1))
                bc[cs.off + (long long)(gy >> 1) * cs.nx + (gx >> 1)] = mg_restrict<T>(a, b, c);
        });
}

// Up: x = xs + P x_c, r = b - L x, x += S(r).  FINAL: x is chi2 of step 3 and step 4 follows,
// z = x1 - (x2 - chi2 / sqrt(dt)) / sqrt(kappa).
template <typename T, bool FINAL>
__global__ __launch_bounds__(kMgRegThreads) void k_mg_up2d(const Sys* sys, const Sys* csys, const int* mask, const cx<T>* b,
                                                          const cx<T>* xs, const cx<T>* xc, cx<T>* x, const cx<T>* x1,
                                                          const cx<T>* x2, cx<T>* z, int nu, int halo) {
    __shared__ cx<T> edges[2][kMgNW][2][kTX];
    const int si = blockIdx.y, wv = (int)threadIdx.x >> 6;
    if (mask && !mask[si]) return;
    const Sys& s = sys[si];
    MgRegion reg;
    if (!reg.init(s, halo)) return;
    using Row = typename RowStencil<T>::Row;
    const RowStencil<T> st(s);
    auto make = [&](cx<T> l, cx<T> c, cx<T> r) { return st.row(l, c, r); };
    int e = 0;
    cx<T> R[kMgNP], D[kMgNP], X[kMgNP];
    {
        const Sys& c = csys[si];
        const cx<T>* xcs = xc + c.off;
        const int cnx = c.nx, cny = c.ny;
        RegionRows g = reg.rows0;
#pragma unroll
        for (int i = 0; i < kMgNP; ++i, g.next()) {
            R[i] = b[g.at()];
            X[i] = xs[g.at()] +
                   mg_interp<T>((int)g.gx, g.gy, cnx, cny, [&](int p, int q) { return xcs[(long long)q * cnx + p]; });
        }
    }
    row_sweep<T, kMgNP, kMgNW>(X, edges[e], wv, make, [&](int i, const Row& p, const Row& q, const Row& w, cx<T>) {
        R[i] = R[i] - st.L(p, q, w);
    });
    e ^= 1;
    const double(*cb)[2] = s.cb[1];
    const T c0 = T(cb[0][0]);
#pragma unroll
    for (int i = 0; i < kMgNP; ++i) {
        D[i] = c0 * R[i];
        X[i] = X[i] + D[i];
    }
    for (int j = 1; j < nu; ++j) {
        const T c1 = T(cb[j][0]), c2 = T(cb[j][1]);
        row_sweep<T, kMgNP, kMgNW>(D, edges[e], wv, make,
                                   [&](int i, const Row& p, const Row& q, const Row& w, cx<T> dB) {
                                       R[i] = R[i] - st.L(p, q, w);
                                       D[i] = c1 * dB + c2 * R[i];
                                       X[i] = X[i] + D[i];
                                   });
        e ^= 1;
    }
    RegionRows g = reg.rows0;
#pragma unroll
    for (int i = 0; i < kMgNP; ++i, g.next())
        if (reg.owned(i)) {
            const long long gi = g.at();
            x[gi] = X[i];
            if constexpr (FINAL) z[gi] = x1[gi] - T(s.isq_kap) * (x2[gi] - T(s.isq_dt) * X[i]);
        }
}

// The levels of at most 64 x 64 nodes, one workgroup per system: down to the coarsest level (its Chebyshev
// solve included) and up again, each vector in the registers of the threads (four consecutive rows of one
// column each), stencils through LDS with one barrier.  x and b of the levels above the coarsest wait in their
// global buffers, read back by the thread that wrote them.
constexpr int kMgTail = 4, kMgTailThreads = 1024, kMgTailRows = 4;
template <typename T>
struct MgTailLevels {
    int n;                          // levels, the last one the coarsest
    const Sys* sys[kMgTail];
    cx<T>* x[kMgTail];
    cx<T>* b[kMgTail];              // b[0]: the right-hand side
};

template <typename T>
__global__ __launch_bounds__(kMgTailThreads) void k_mg_tail(const MgTailLevels<T> lev, const int* mask, int nu,
                                                           int coarse_its) {
    __shared__ cx<T> buf[2][kTX * kTX];
    const int si = blockIdx.x;
    if (mask && !mask[si]) return;
    const int x = (int)threadIdx.x & 63, y0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) * kMgTailRows;
    using Row = typename RowStencil<T>::Row;
    int set = 0;
    // u into LDS (all rows of the level), visible after the barrier; two buffers in turn
    auto stage = [&](const cx<T> (&u)[kMgTailRows], int nx, int ny) -> const cx<T>* {
        cx<T>* p = buf[set];
        set ^= 1;
#pragma unroll
        for (int i = 0; i < kMgTailRows; ++i)
            if (x < nx && y0 + i < ny) p[(y0 + i) * kTX + x] = u[i];
        __syncthreads();
        return p;
    };
    // R = B - L u
    auto residual = [&](const Sys& s, const RowStencil<T>& st, const cx<T> (&B)[kMgTailRows], const cx<T> (&u)[kMgTailRows],
                        cx<T> (&R)[kMgTailRows]) {
        const int nx = s.nx, ny = s.ny;
        const cx<T>* p = stage(u, nx, ny);
        if (y0 >= ny || x >= nx) return;
        const int xl = x == 0 ? nx - 1 : x - 1, xr = x == nx - 1 ? 0 : x + 1;
        Row A{}, C{};
#pragma unroll
        for (int a = 0; a < kMgTailRows + 2; ++a) {
            int y = y0 - 1 + a;
            y = y < 0 ? ny - 1 : y >= ny ? y - ny : y;
            const cx<T>* row = p + y * kTX;
            const Row N = st.row(row[xl], row[x], row[xr]);
            if (a >= 2) R[a - 2] = B[a - 2] - st.L(A, C, N);
            A = C;
            C = N;
        }
    };
    cx<T> B[kMgTailRows], R[kMgTailRows], D[kMgTailRows], X[kMgTailRows];
    auto inside = [&](const Sys& s, int i) { return x < s.nx && y0 + i < s.ny; };
    auto node = [&](const Sys& s, int i) { return s.off + (long long)(y0 + i) * s.nx + x; };
#pragma unroll
    for (int i = 0; i < kMgTailRows; ++i) {
        B[i] = cx<T>{T(0), T(0)};
        if (inside(lev.sys[0][si], i)) B[i] = lev.b[0][node(lev.sys[0][si], i)];
    }
    // Chebyshev iterations 1 .. its - 1 on R, D, X
    auto smooth = [&](const Sys& s, const RowStencil<T>& st, int its) {
        for (int j = 1; j < its; ++j) {
            residual(s, st, R, D, R);
            const T c1 = T(s.cb[1][j][0]), c2 = T(s.cb[1][j][1]);
#pragma unroll
            for (int i = 0; i < kMgTailRows; ++i) {
                D[i] = c1 * D[i] + c2 * R[i];
                X[i] = X[i] + D[i];
            }
        }
    };
    // from zero: R = B, D = X = c0 B
    auto start = [&](const Sys& s) {
        const T c0 = T(s.cb[1][0][0]);
#pragma unroll
        for (int i = 0; i < kMgTailRows; ++i) {
            R[i] = B[i];
            D[i] = c0 * B[i];
            X[i] = D[i];
        }
    };
    for (int l = 0; l + 1 < lev.n; ++l) {
        const Sys& s = lev.sys[l][si];
        const Sys& c = lev.sys[l + 1][si];
        const RowStencil<T> st(s);
        start(s);
        smooth(s, st, nu);
#pragma unroll
        for (int i = 0; i < kMgTailRows; ++i)
            if (inside(s, i)) {
                lev.x[l][node(s, i)] = X[i];
                if (l > 0) lev.b[l][node(s, i)] = B[i];
            }
        residual(s, st, B, X, R);
        // restriction: coarse node (x, y0 + i) from the fine nodes around (2 x, 2 (y0 + i))
        const int fnx = s.nx, fny = s.ny;
        const cx<T>* p = stage(R, fnx, fny);
#pragma unroll
        for (int i = 0; i < kMgTailRows; ++i) {
            B[i] = cx<T>{T(0), T(0)};
            if (!inside(c, i)) continue;
            const int fx = 2 * x, fy = 2 * (y0 + i), xl = fx == 0 ? fnx - 1 : fx - 1, yl = fy == 0 ? fny - 1 : fy - 1;
            auto raw = [&](int y) { return Raw<T>{p[y * kTX + xl], p[y * kTX + fx], p[y * kTX + fx + 1]}; };
            B[i] = mg_restrict<T>(raw(yl), raw(fy), raw(fy + 1));
        }
    }
    {
        const Sys& s = lev.sys[lev.n - 1][si];
        start(s);
        smooth(s, RowStencil<T>(s), coarse_its);
    }
    for (int l = lev.n - 2; l >= 0; --l) {
        const Sys& s = lev.sys[l][si];
        const int cnx = lev.sys[l + 1][si].nx, cny = lev.sys[l + 1][si].ny;
        const RowStencil<T> st(s);
        const cx<T>* p = stage(X, cnx, cny);
#pragma unroll
        for (int i = 0; i < kMgTailRows; ++i) {
            X[i] = B[i] = R[i] = cx<T>{T(0), T(0)};
            if (!inside(s, i)) continue;
            X[i] = lev.x[l][node(s, i)] + mg_interp<T>(x, y0 + i, cnx, cny, [&](int a, int b) { return p[b * kTX + a]; });
            B[i] = lev.b[l][node(s, i)];
        }
        residual(s, st, B, X, R);
        const T c0 = T(s.cb[1][0][0]);
#pragma unroll
        for (int i = 0; i < kMgTailRows; ++i) {
            D[i] = c0 * R[i];
            X[i] = X[i] + D[i];
        }
        smooth(s, st, nu);
    }
    const Sys& s = lev.sys[0][si];
#pragma unroll
    for (int i = 0; i < kMgTailRows; ++i)
        if (inside(s, i)) lev.x[0][node(s, i)] = X[i];
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
// smoothing on one level: from zero (ADD = false, b given) or as a correction from the residual r
// (ADD = true); nu Chebyshev iterations in all
template <int DIM, int TY, typename T, bool ADD>
static void mg_smooth(const Dev& d, int nu, const cx<T>* b, cx<T>* r, cx<T>* d0, cx<T>* d1, cx<T>* x, const int* mask,
                      hipStream_t st) {
    {
        // reads b or r (and x when ADD), writes r or d, d and x
        ProbeScope ps(d, KID_MG, st, (double)d.NT * sizeof(cx<T>) * (ADD ? 4.0 : 4.0), mask);
        hipLaunchKernelGGL((k_mg_start<DIM, TY, T, ADD>), TILE_GRID, d.sys, d.tiles, mask, b, r, d0, x);
    }
    cx<T>* D[2] = {d0, d1};
    for (int j = 1; j < nu; ++j) {
        const bool last = j == nu - 1;
        ProbeScope ps(d, KID_MG, st, (double)d.NT * sizeof(cx<T>) * (last ? 4.0 : 6.0), mask);
        if (last)
            hipLaunchKernelGGL((k_mg_iter<DIM, TY, T, true>), TILE_GRID, d.sys, d.tiles, mask, j, D[(j - 1) & 1],
                               D[j & 1], r, x);
        else
            hipLaunchKernelGGL((k_mg_iter<DIM, TY, T, false>), TILE_GRID, d.sys, d.tiles, mask, j, D[(j - 1) & 1],
                               D[j & 1], r, x);
    }
}

// The fused 2D cycle: its first level of at most 64 x 64 nodes in every system, or -1 (3D, many smoothing
// iterations, a coarsest level above 64 x 64).
int mg_tail_level(const Dev& fine, const MgLevels& mg) {
    if (fine.dim != 2 || mg.nu > kMgFusedNu) return -1;
    for (int l = 0; l <= mg.n; ++l)
        if ((fine.maxn[0] >> l) <= kTX && (fine.maxn[1] >> l) <= kTX) return mg.n - l < kMgTail ? l : -1;
    return -1;
}

// x = V(b); rhs 1 and 2: the fine level's b is formed from src (k_mg_down2d), with a tail below the fine level.
// xs: work vector of the fine level.  x1 and x2 set: step 4 as well.
template <typename T>
void launch_mg_fused2d(const Dev& fine, const MgLevels& mg, int tail, int rhs, const cx<T>* v, const cx<T>* src, cx<T>* b,
                       cx<T>* x, cx<T>* xs, const cx<T>* x1, const cx<T>* x2, cx<T>* z, const int* mask, hipStream_t st) {
    auto dev = [&](int l) -> const Dev& { return l == 0 ? fine : mg.lev[l - 1]; };
    auto B = [&](int l) { return l == 0 ? b : (cx<T>*)mg.b[l - 1]; };
    auto X = [&](int l) { return l == 0 ? x : (cx<T>*)mg.x[l - 1]; };
    auto XS = [&](int l) { return l == 0 ? xs : (cx<T>*)mg.r[l - 1]; };
    auto grid = [&](int l, int halo) {
        const int IX = kTX - 2 * halo, IY = kMgRegY - 2 * halo;
        const int nx = fine.maxn[0] >> l, ny = fine.maxn[1] >> l;
        return dim3(((nx + IX - 1) / IX) * ((ny + IY - 1) / IY), fine.S);
    };
    const double cb = sizeof(cx<T>);
    for (int l = 0; l < tail; ++l) {
        const Dev& d = dev(l);
        const int form = l == 0 ? rhs : 0, halo = mg.nu + 1 + (form ? 1 : 0);
        ProbeScope ps(d, KID_MG, st, (double)d.NT * cb * (form == 0 ? 2.25 : form == 1 ? 4.25 : 3.25), mask);
        auto go = [&](auto rc) {
            hipLaunchKernelGGL((k_mg_down2d<T, decltype(rc)::value>), grid(l, halo), dim3(kMgRegThreads), 0, st, d.sys,
                               dev(l + 1).sys, mask, v, form ? src : (const cx<T>*)B(l), B(l), XS(l), B(l + 1), mg.nu,
                               halo);
        };
        if (form == 1) go(std::integral_constant<int, 1>{});
        else if (form == 2) go(std::integral_constant<int, 2>{});
        else go(std::integral_constant<int, 0>{});
    }
    {
        const Dev& d = dev(tail);
        MgTailLevels<T> t{};
        t.n = mg.n + 1 - tail;
        for (int l = 0; l < t.n; ++l) {
            t.sys[l] = dev(tail + l).sys;
            t.x[l] = X(tail + l);
            t.b[l] = B(tail + l);
        }
        ProbeScope ps(d, KID_MG, st, (double)d.NT * cb * 4.0, mask);
        hipLaunchKernelGGL(k_mg_tail<T>, dim3(d.S), dim3(kMgTailThreads), 0, st, t, mask, mg.nu, mg.coarse_its);
    }
    for (int l = tail - 1; l >= 0; --l) {
        const Dev& d = dev(l);
        const bool fin = l == 0 && x1;
        ProbeScope ps(d, KID_MG, st, (double)d.NT * cb * (fin ? 6.25 : 3.25), mask);
        auto go = [&](auto fc) {
            hipLaunchKernelGGL((k_mg_up2d<T, decltype(fc)::value>), grid(l, mg.nu), dim3(kMgRegThreads), 0, st, d.sys,
                               dev(l + 1).sys, mask, (const cx<T>*)B(l), (const cx<T>*)XS(l), (const cx<T>*)X(l + 1), X(l),
                               x1, x2, z, mg.nu, mg.nu);
        };
        if (fin) go(std::true_type{});
        else go(std::false_type{});
    }
}
template void launch_mg_fused2d<double>(const Dev&, const MgLevels&, int, int, const zd*, const zd*, zd*, zd*, zd*,
                                        const zd*, const zd*, zd*, const int*, hipStream_t);
template void launch_mg_fused2d<float>(const Dev&, const MgLevels&, int, int, const zf*, const zf*, zf*, zf*, zf*,
                                       const zf*, const zf*, zf*, const int*, hipStream_t);

template <typename T>
void launch_mg_vcycle(const Dev& fine, const MgLevels& mg, const cx<T>* b, cx<T>* x, cx<T>* r, cx<T>* d0, cx<T>* d1,
                      const int* mask, hipStream_t st) {
    // level l: 0 = the fine level (the caller's buffers and tiles), 1..mg.n the coarser ones
    const int L = mg.n + 1;
    auto dev = [&](int l) -> const Dev& { return l == 0 ? fine : mg.lev[l - 1]; };
    auto B = [&](int l) { return l == 0 ? const_cast<cx<T>*>(b) : (cx<T>*)mg.b[l - 1]; };
    auto X = [&](int l) { return l == 0 ? x : (cx<T>*)mg.x[l - 1]; };
    auto R = [&](int l) { return l == 0 ? r : (cx<T>*)mg.r[l - 1]; };
    auto D0 = [&](int l) { return l == 0 ? d0 : (cx<T>*)mg.d0[l - 1]; };
    auto D1 = [&](int l) { return l == 0 ? d1 : (cx<T>*)mg.d1[l - 1]; };
    // down: smooth, residual, restrict
    for (int l = 0; l + 1 < L; ++l) {
        const Dev& d = dev(l);
        const Dev& dc = dev(l + 1);
        dispatch(d, [&](auto Dc, auto TYc) {
            constexpr int DIM = Dc(), TY = TYc();
            mg_smooth<DIM, TY, T, false>(d, mg.nu, B(l), R(l), D0(l), D1(l), X(l), mask, st);
            ProbeScope ps(d, KID_MG, st, (double)d.NT * sizeof(cx<T>) * 3.0, mask);
            hipLaunchKernelGGL((k_mg_residual<DIM, TY, T>), dim3(d.ntiles), dim3(kBlock), 0, st, d.sys, d.tiles, mask,
                               B(l), X(l), R(l));
        });
        dispatch(dc, [&](auto Dc, auto TYc) {
            constexpr int DIM = Dc(), TY = TYc();
            ProbeScope ps(dc, KID_MG, st, (double)dc.NT * sizeof(cx<T>) * (DIM == 3 ? 9.0 : 5.0), mask);
            hipLaunchKernelGGL((k_mg_restrict<DIM, TY, T>), dim3(dc.ntiles), dim3(kBlock), 0, st, dc.sys, dc.tiles,
                               mask, d.sys, R(l), B(l + 1));
        });
    }
    // coarsest level
    {
        const Dev& d = dev(L - 1);
        ProbeScope ps(d, KID_MG, st, (double)d.NT * sizeof(cx<T>) * 2.0, mask);
        if (d.dim == 3)
            hipLaunchKernelGGL((k_mg_coarse<3, T>), dim3(d.S), dim3(kMgThreads), 0, st, d.sys, mask, mg.coarse_its,
                               B(L - 1), X(L - 1));
        else
            hipLaunchKernelGGL((k_mg_coarse<2, T>), dim3(d.S), dim3(kMgThreads), 0, st, d.sys, mask, mg.coarse_its,
                               B(L - 1), X(L - 1));
    }
    // up: prolong, residual, smooth the correction
    for (int l = L - 2; l >= 0; --l) {
        const Dev& d = dev(l);
        const Dev& dc = dev(l + 1);
        dispatch(d, [&](auto Dc, auto TYc) {
            constexpr int DIM = Dc(), TY = TYc();
            {
                ProbeScope ps(d, KID_MG, st, (double)d.NT * sizeof(cx<T>) * (2.0 + 1.0 / (1 << DIM)), mask);
                hipLaunchKernelGGL((k_mg_prolong<DIM, TY, T>), dim3(d.ntiles), dim3(kBlock), 0, st, d.sys, d.tiles,
                                   mask, dc.sys, X(l + 1), X(l));
            }
            {
                ProbeScope ps(d, KID_MG, st, (double)d.NT * sizeof(cx<T>) * 3.0, mask);
                hipLaunchKernelGGL((k_mg_residual<DIM, TY, T>), dim3(d.ntiles), dim3(kBlock), 0, st, d.sys, d.tiles,
                                   mask, B(l), X(l), R(l));
            }
            mg_smooth<DIM, TY, T, true>(d, mg.nu, nullptr, R(l), D0(l), D1(l), X(l), mask, st);
        });
    }
}
template void launch_mg_vcycle<double>(const Dev&, const MgLevels&, const zd*, zd*, zd*, zd*, zd*, const int*,
                                       hipStream_t);
template void launch_mg_vcycle<float>(const Dev&, const MgLevels&, const zf*, zf*, zf*, zf*, zf*, const int*,
                                      hipStream_t);

}  // namespace apfc
