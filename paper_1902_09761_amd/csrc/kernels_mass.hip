// The mass matrix's inverse on the uniform periodic mesh, for gfx950: step 1 of the block preconditioner
// (Eq. (12), M x1 = beta1) by a separable approximate inverse, and the auxiliary field zeta = M^{-1} G eta to
// FP64 rounding by one line filter per direction, with their launchers.
#include "kernels_common.h"

#include <algorithm>

namespace apfc {

// On the uniform periodic mesh the Q1 mass matrix is the Kronecker product of the 1D matrices
// (h/6) tridiag(1, 4, 1) of the directions, so its inverse is the Kronecker product of their inverses.
// The 1D inverse has the entries (sqrt(3)/h) rho^|k| with rho = sqrt(3) - 2, which fall by |rho| ~ 0.27
// per node; W keeps |k| <= R in each direction, so x1 = W beta1 is one 1D filter of 2R + 1 taps per
// direction (Sys::wsep holds (sqrt(3)/h) rho^k).  Taps that wrap onto the same node of a short periodic
// direction add up.
//
// A workgroup of 512 threads owns a brick of 64 x kMassBY nodes per plane and BZ planes (one plane in
// 2D).  Each plane, from R planes before the brick to R planes after it (periodic), passes through three
// stages: its region of (64 + 2R) x (kMassBY + 2R) nodes is staged in LDS (the next plane's loads in flight
// meanwhile); the region's rows are filtered in x into a second LDS array; that is filtered in y at the thread's
// node, where the last 2R + 1 such values of the column stay in registers for the z filter.  A phase between
// two barriers takes one plane in each stage, on two buffers per array: one barrier per plane and three
// independent pieces of work in it, where stage after stage took three barriers per plane and their latency
// bounded the kernel (75 x 66 x 58 x 7 in FP64: 62.8 us, now 51.9; 128^3 x 6 in FP32, where the LDS reads bound it: 72.4 us, now 71.7).
// HBM traffic: beta1 read once (the halos come from L2) and x1 written once; about 4 (2D) and 7 (3D)
// multiply-adds per tap and node.
__device__ __forceinline__ int wrapm(int g, int n) {
    g %= n;
    return g < 0 ? g + n : g;
}

template <int DIM, int BZ, typename T, int R>
__global__ __launch_bounds__(kMassThreads) void k_mass_sep(const Sys* sys, const Tile* tiles, const int* mask,
                                                          const cx<T>* __restrict__ v, cx<T>* __restrict__ x1) {
    constexpr int PX = kTX + 2 * R, PY = kMassBY + 2 * R, PP = PX * PY;
    constexpr int NZ = DIM == 3 ? BZ + 2 * R : 1;   // planes marched
    static_assert(kMassThreads == kTX * kMassBY, "one thread per node of a brick plane");
    constexpr int NS = (PP + kMassThreads - 1) / kMassThreads;   // staged nodes per thread and plane
    __shared__ cx<T> bufA[2][PP];
    __shared__ cx<T> bufB[2][PY * kTX];
    const Tile tile = tiles[blockIdx.x];
    if (mask && !mask[tile.sys]) return;
    const Sys* sp = sys + tile.sys;
    const int nx = sp->nx, ny = sp->ny, nz = sp->nz;
    const long long off = sp->off, plane = (long long)nx * ny;
    T w[R + 1];
#pragma unroll
    for (int k = 0; k <= R; ++k) w[k] = T(sp->wsep[k]);
    const int t = (int)threadIdx.x, lx = t % kTX, ly = t / kTX;
    static_assert(NS <= 3, "at most three staged nodes per thread");
    // the thread's staged nodes t, t + 512, t + 1024 of a plane region (offsets inside the plane)
    auto goff = [&](int e) -> long long {
        const int gx = wrapm(tile.x0 - R + e % PX, nx), gy = wrapm(tile.y0 - R + e / PX, ny);
        return e < PP ? (long long)gy * nx + gx : 0;
    };
    const long long o0 = goff(t), o1 = NS > 1 ? goff(t + kMassThreads) : 0, o2 = NS > 2 ? goff(t + 2 * kMassThreads) : 0;
    const bool h1 = NS > 1 && t + kMassThreads < PP, h2 = NS > 2 && t + 2 * kMassThreads < PP;
    const cx<T> zero{T(0), T(0)};
    int zz = DIM == 3 ? wrapm(tile.z - R, nz) : 0;
    cx<T> a0 = zero, a1 = zero, a2 = zero;
    auto fetch = [&](long long base) {   // nodes past the region: the plane's first node, not used
        a0 = v[base + o0];
        if constexpr (NS > 1) a1 = v[base + o1];
        if constexpr (NS > 2) a2 = v[base + o2];
    };
    fetch(off + zz * plane);
    cx<T> Q[2 * R + 1];
#pragma unroll
    for (int i = 0; i < 2 * R + 1; ++i) Q[i] = zero;
    const int x = tile.x0 + lx, y = tile.y0 + ly;
    // phase p: plane p into bufA[p & 1]; plane p - 1 filtered in x from bufA[(p - 1) & 1] into bufB[(p - 1) & 1];
    // plane p - 2 filtered in y from bufB[p & 1]
#pragma unroll 1
    for (int p = 0; p < NZ + 2; ++p) {
        cx<T>* A = bufA[p & 1];
        if (p < NZ) {
            A[t] = a0;
            if (h1) A[t + kMassThreads] = a1;
            if (h2) A[t + 2 * kMassThreads] = a2;
            if (p + 1 < NZ) {
                zz = zz + 1 == nz ? 0 : zz + 1;
                fetch(off + zz * plane);
            }
        }
        if (p >= 1 && p <= NZ) {
            // x filter of every region row at the 64 brick columns
            const cx<T>* Ap = bufA[(p - 1) & 1];
            cx<T>* B = bufB[(p - 1) & 1];
            for (int e = t; e < PY * kTX; e += kMassThreads) {
                const cx<T>* row = Ap + (e / kTX) * PX + (e % kTX) + R;
                cx<T> acc = w[0] * row[0];
#pragma unroll
                for (int k = 1; k <= R; ++k) acc = acc + w[k] * (row[-k] + row[k]);
                B[e] = acc;
            }
        }
        if (p >= 2) {
            // y filter at the thread's node
            const cx<T>* col = bufB[p & 1] + (ly + R) * kTX + lx;
            cx<T> u = w[0] * col[0];
#pragma unroll
            for (int k = 1; k <= R; ++k) u = u + w[k] * (col[-k * kTX] + col[k * kTX]);
            if constexpr (DIM == 2) {
                if (x < nx && y < ny) x1[off + (long long)y * nx + x] = u;
            } else {
                // Q[i] holds the filtered plane tile.z - 3R + p - 2 + i; the z filter is centred on Q[R]
#pragma unroll
                for (int i = 0; i < 2 * R; ++i) Q[i] = Q[i + 1];
                Q[2 * R] = u;
                const int z = tile.z + p - 2 - 2 * R;
                if (p - 2 >= 2 * R && x < nx && y < ny && z < nz) {
                    cx<T> o = w[0] * Q[R];
#pragma unroll
                    for (int k = 1; k <= R; ++k) o = o + w[k] * (Q[R - k] + Q[R + k]);
                    x1[off + ((long long)z * ny + y) * nx + x] = o;
                }
            }
        }
        __syncthreads();
    }
}

template <typename T>
void launch_mass_sep(const Dev& d, int R, const cx<T>* v, cx<T>* x1, const int* mask, hipStream_t st) {
    ProbeScope ps(d, KID_MASS, st, (double)d.NT * 2.0 * sizeof(cx<T>), mask, true);
    auto go = [&](auto rc) {
        constexpr int RR = decltype(rc)::value;
        if (d.dim == 3)
            brick_depth(d, [&](auto bz) {
                ps.launch(k_mass_sep<3, decltype(bz)::value, T, RR>, dim3(d.nmtiles), dim3(kMassThreads), d.sys,
                          d.mtiles, mask, v, x1);
            });
        else
            ps.launch(k_mass_sep<2, 1, T, RR>, dim3(d.nmtiles), dim3(kMassThreads), d.sys, d.mtiles, mask, v, x1);
    };
    static_assert(kMassRMax == 4, "one case per tap count");
    switch (R) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        default: go(std::integral_constant<int, 4>{}); break;
    }
}
template void launch_mass_sep<double>(const Dev&, int, const zd*, zd*, const int*, hipStream_t);
template void launch_mass_sep<float>(const Dev&, int, const zf*, zf*, const int*, hipStream_t);

// ------------------------------------------------------------------------------------------
// zeta_j = M^{-1} G_j eta_j (the auxiliary field of Algorithm 1, the energy and its gradient) to FP64 rounding.
//
// With the 1D matrices m = (h/6) P, P = [1 4 1], k = (1/h) Q, Q = [-1 2 -1], d = E/2, E = [-1 0 1] of the
// directions, M = m (x) m (x) m, so M^{-1} G_j = sum_dir P_dir^{-1} (-(6/h^2) Q_dir + i (6 k_{j,dir}/h) E_dir):
// the other directions' mass factors cancel, and zeta is the sum of one line filter per direction.  P^{-1} on
// a line has the entries rho^|n|/(2 sqrt 3), rho = sqrt 3 - 2; with |rho|^kLineHalo < 1e-17 the line solve is
// a causal and an anticausal first-order recursion c+_i = y_i + rho c+_{i-1}, c-_i = y_i + rho c-_{i+1},
// P^{-1} y = (c+ + c- - y)/(2 sqrt 3), each started kLineHalo nodes before its first output (periodic
// images of a short line included).  Bound by memory: three (2D: two) passes over eta and zeta.  Solving for
// M by 100 (2D: 60) Chebyshev iterations to the same error, a launch and six vectors each, took apfc_energy of
// 1024^2 x 3 to 2736 us (145 us with the filters) and, with the nodal part of the gradient formed once per
// amplitude, apfc_energy_grad of 90 x 96 x 77 x 6 to 7618 us (358 us).
// ------------------------------------------------------------------------------------------
constexpr int kLineHalo = 32;
constexpr double kRho = -0.26794919243112270647;        // sqrt(3) - 2
constexpr double kLineNorm = 0.28867513459481288225;    // 1/(2 sqrt 3)

// x: a wave holds 64 blocks of 8 consecutive nodes, whole line segments (output nodes plus kLineHalo on either
// side) packed one after the other (gpw of them per wave, so that short lines leave few lanes idle).  A lane
// runs both recursions over its block and takes the rest of the recursion from the four neighbouring lanes'
// block sums (rho^32 of anything further away is below rounding); global loads and stores are coalesced
// through LDS (blocks padded by one node against bank conflicts).
constexpr int kLineB = 8, kLineMax = 64 * kLineB - 2 * kLineHalo;

__device__ __forceinline__ int line_segs(int n) { return (n + kLineMax - 1) / kLineMax; }

// The system of this workgroup, which of the system's workgroups it is and how many there are: row blockIdx.y of the
// grid, or with tiles the one of tile blockIdx.x (launch_zeta).
struct ZetaBlock {
    const Sys* s;
    int b, n;
    __device__ ZetaBlock(const Sys* sys, const Tile* tiles) {
        s = sys + (tiles ? tiles[blockIdx.x].sys : (int)blockIdx.y);
        b = (int)blockIdx.x - (tiles ? s->tbeg : 0);
        n = tiles ? s->tend - s->tbeg : (int)gridDim.x;
    }
};

__global__ __launch_bounds__(kBlock) void k_zeta_x(const Sys* sys, const Tile* tiles, const zd* __restrict__ eta,
                                                  zd* __restrict__ zeta) {
    __shared__ zd buf[kBlock / 64][64 * (kLineB + 1)];
    const ZetaBlock blk(sys, tiles);
    const Sys* s = blk.s;
    const int nx = s->nx, segs = line_segs(nx), nout = (nx + segs - 1) / segs;
    const int gw = (nout + 2 * kLineHalo + kLineB - 1) / kLineB, gpw = 64 / gw, gn = gw * kLineB;
    const long long off = s->off, items = (long long)s->ny * s->nz * segs;
    const int wv = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const double a = -6.0 / (s->h * s->h) * kLineNorm, b = 6.0 * s->kv[0] / s->h * kLineNorm;
    auto slot = [](int e) { return e + e / kLineB; };
    zd* w = buf[wv];
    // no neighbour inside the segment: the block's own end stands in, kLineHalo nodes from any output
    const bool first = lane % gw == 0, last = lane % gw == gw - 1 || lane == 63;
    const double rb = kRho * kRho, rho8 = rb * rb * rb * rb;
    for (long long it0 = (long long)blk.b * 4 * gpw; it0 < items; it0 += (long long)blk.n * 4 * gpw) {
        auto node = [&](int e, bool& out) -> long long {   // node of element e, -1: none; out: an output node
            const int g = e / gn, p = e - g * gn;
            const long long item = it0 + (long long)wv * gpw + g;
            out = false;
            if (g >= gpw || item >= items) return -1;
            const long long row = item / segs;
            const int xs = (int)(item - row * segs) * nout;
            int x = (xs - kLineHalo + p) % nx;
            x = x < 0 ? x + nx : x;
            out = p >= kLineHalo && p < kLineHalo + nout && xs - kLineHalo + p < nx;
            return off + row * nx + x;
        };
        bool out[kLineB];
        long long idx[kLineB];
#pragma unroll
        for (int i = 0; i < kLineB; ++i) {
            const int e = i * 64 + lane;
            idx[i] = node(e, out[i]);
            w[slot(e)] = idx[i] >= 0 ? eta[idx[i]] : zd{0.0, 0.0};
        }
        __syncthreads();
        zd u[kLineB + 2];
        u[0] = w[slot(first ? lane * kLineB : lane * kLineB - 1)];
#pragma unroll
        for (int k = 0; k < kLineB; ++k) u[k + 1] = w[slot(lane * kLineB + k)];
        u[kLineB + 1] = w[slot(last ? lane * kLineB + kLineB - 1 : (lane + 1) * kLineB)];
        zd y[kLineB], f[kLineB], c[kLineB];
#pragma unroll
        for (int k = 0; k < kLineB; ++k)
            y[k] = a * ((u[k + 1] + u[k + 1]) - (u[k] + u[k + 2])) + b * mul_i(u[k + 2] - u[k]);
        f[0] = y[0];
        c[kLineB - 1] = y[kLineB - 1];
#pragma unroll
        for (int k = 1; k < kLineB; ++k) {
            f[k] = y[k] + kRho * f[k - 1];
            c[kLineB - 1 - k] = y[kLineB - 1 - k] + kRho * c[kLineB - k];
        }
        zd cf{0.0, 0.0}, cb{0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            cf = lane_shift<kDppWaveShr1>(f[kLineB - 1] + rho8 * cf);
            cb = lane_shift<kDppWaveShl1>(c[0] + rho8 * cb);
        }
        double pw[kLineB + 1];
        pw[0] = 1.0;
#pragma unroll
        for (int k = 1; k <= kLineB; ++k) pw[k] = pw[k - 1] * kRho;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kLineB; ++k)
            w[slot(lane * kLineB + k)] = ((f[k] + pw[k + 1] * cf) + (c[k] + pw[kLineB - k] * cb)) - y[k];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kLineB; ++i)
            if (out[i]) zeta[idx[i]] = w[slot(i * 64 + lane)];
        __syncthreads();
    }
}

// y (DIR = 1) and z (DIR = 2), zeta += the direction's filter of eta: a thread takes kLineSeg consecutive nodes of
// one line, lanes along x.  It walks down to them from kLineHalo nodes before, keeping c+ of its outputs in
// registers, and back up from kLineHalo nodes after; the re-read nodes come from L2.
constexpr int kLineSeg = 32;

template <int DIR>
__global__ __launch_bounds__(kBlock) void k_zeta_line(const Sys* sys, const Tile* tiles, const zd* __restrict__ eta,
                                                     zd* __restrict__ zeta) {
    const ZetaBlock blk(sys, tiles);
    const Sys* s = blk.s;
    const int n = DIR == 1 ? s->ny : s->nz, nx = s->nx;
    const int lines = DIR == 1 ? nx * s->nz : nx * s->ny, segs = (n + kLineSeg - 1) / kLineSeg;
    const long long stride = DIR == 1 ? nx : (long long)nx * s->ny;
    const double a = -6.0 / (s->h * s->h) * kLineNorm, b = 6.0 * s->kv[DIR] / s->h * kLineNorm;
    auto wrap = [&](int p) {
        p %= n;
        return p < 0 ? p + n : p;
    };
    auto src = [&](zd l, zd c, zd r) { return a * ((c + c) - (l + r)) + b * mul_i(r - l); };
    for (long long t = (long long)blk.b * kBlock + threadIdx.x; t < (long long)lines * segs; t += (long long)blk.n * kBlock) {
        const int seg = (int)(t / lines), line = (int)(t - (long long)seg * lines);
        const long long base = s->off + (DIR == 1 ? (long long)(line / nx) * nx * s->ny + line % nx : (long long)line);
        const zd* e = eta + base;
        zd* z = zeta + base;
        const int s0 = seg * kLineSeg;
        zd f[kLineSeg], v{0.0, 0.0};
        {
            int p = wrap(s0 - kLineHalo - 1);
            auto next = [&]() {
                const zd u = e[p * stride];
                p = p + 1 == n ? 0 : p + 1;
                return u;
            };
            zd l = next(), c = next();
#pragma unroll 8
            for (int k = 0; k < kLineHalo; ++k) {
                const zd r = next();
                v = src(l, c, r) + kRho * v;
                l = c;
                c = r;
            }
#pragma unroll
            for (int k = 0; k < kLineSeg; ++k) {
                const zd r = next();
                v = src(l, c, r) + kRho * v;
                f[k] = v;
                l = c;
                c = r;
            }
        }
        v = zd{0.0, 0.0};
        int p = wrap(s0 + kLineSeg + kLineHalo);
        auto prev = [&]() {
            const zd u = e[p * stride];
            p = p == 0 ? n - 1 : p - 1;
            return u;
        };
        zd r = prev(), c = prev();
#pragma unroll 8
        for (int k = 0; k < kLineHalo; ++k) {
            const zd l = prev();
            v = src(l, c, r) + kRho * v;
            r = c;
            c = l;
        }
#pragma unroll
        for (int k = kLineSeg - 1; k >= 0; --k) {
            const zd l = prev();
            const zd y = src(l, c, r);
            v = y + kRho * v;
            if (s0 + k < n) {
                const long long o = (s0 + k) * stride;
                z[o] = z[o] + ((f[k] + v) - y);
            }
            r = c;
            c = l;
        }
    }
}

// Grid: the workgroups that the largest mesh needs for every system, where the meshes are of like size; else the stencil
// tiles, each system's sharing out its lines (a few more workgroups than lines: apfc_energy_grad of one
// 90 x 96 x 77 x 6 in 385 us instead of 356).  With 1024^2 and 1023 meshes of 16^2, x 3, the former is nearly all empty
// workgroups (apfc_energy 4903 us, by tiles 268); the line lies where half of the larger grid would be empty.
void launch_zeta(const Dev& d, const zd* eta, zd* zeta, hipStream_t st) {
    const int* mx = d.maxn;
    const Tile* tiles = (double)mx[0] * mx[1] * mx[2] * d.S > 2.0 * (double)d.NT ? d.tiles : nullptr;
    auto grid = [&](long long n) { return tiles ? dim3(d.ntiles) : dim3((unsigned)n, d.S); };
    const int segs = (mx[0] + kLineMax - 1) / kLineMax, nout = (mx[0] + segs - 1) / segs;
    const int gpw = 64 / ((nout + 2 * kLineHalo + kLineB - 1) / kLineB);
    const long long rows = (long long)mx[1] * mx[2] * segs;
    hipLaunchKernelGGL(k_zeta_x, grid(std::min<long long>((rows + 4 * gpw - 1) / (4 * gpw), 1 << 20)), dim3(kBlock), 0, st,
                       d.sys, tiles, eta, zeta);
    auto line_blocks = [&](int lines, int n) {
        return ((long long)lines * ((n + kLineSeg - 1) / kLineSeg) + kBlock - 1) / kBlock;
    };
    hipLaunchKernelGGL(k_zeta_line<1>, grid(line_blocks(mx[0] * mx[2], mx[1])), dim3(kBlock), 0, st, d.sys, tiles, eta,
                       zeta);
    if (d.dim == 3)
        hipLaunchKernelGGL(k_zeta_line<2>, grid(line_blocks(mx[0] * mx[1], mx[2])), dim3(kBlock), 0, st, d.sys, tiles,
                           eta, zeta);
}

}  // namespace apfc
