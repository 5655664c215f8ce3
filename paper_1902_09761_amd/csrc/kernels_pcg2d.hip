// The block preconditioner of Eq. (12) with Jacobi-PCG inner solves, fused per step on register-resident
// regions (2D), for gfx950, with its launcher.
#include "kernels_region.h"

namespace apfc {

// ------------------------------------------------------------------------------------------
// Meshes above 64 x 64 nodes, FP64: one launch per CG step.  With the residual r and the direction p = r / D + beta p_old
// a step needs beta = <r, r> / <r_old, r_old> and alpha = (<r, r> / D) / <p, OP p>.  The directions are OP-orthogonal, so
//   <p, OP p> = <r, OP r> / D^2 - beta^2 <p_old, OP p_old>,   1 / alpha = <r, OP r> / (D <r, r>) - beta / alpha_old,
// and both scalars follow from two sums over r alone: a launch takes a whole step (p, x, r) with the sums of the launch
// before it, applies OP to the new r and leaves its two sums, one partial of each per region.  Against 80-bit
// arithmetic a P^{-1} is as accurate as with <p, OP p> summed in a pass of its own (2e-16 rms on amplitude fields).
// Taking a solve's coefficients from the Gram matrix of its Krylov vectors would save launches, but loses up to eight
// digits on smooth right-hand sides, where those vectors are nearly parallel.  The new <r, r> expanded into sums over
// the old r and OP p (one launch per step as well) costs up to 1.4 times the error, where the residual drops fast, and
// 1.4 times the launch with those sums in twice the precision.
//
// A workgroup holds a region of 64 x (NW NP) nodes, interior plus kPcgHalo layers, in registers (row_sweep; one wave
// per NP rows): OP p on the interior and one layer around it (instead of storing it), OP r on the interior.  Launches per
// application of P^{-1}, K steps per solve:
//   PCG_MASS  r = beta1                                              (SEP: x1 given)
//   PCG_STEP  K - 1 times
//   PCG_G     last step's x1; r = beta2 - kappa G x1
//   PCG_STEP  K - 1 times
//   PCG_M     last step's x2; r = M x2
//   PCG_STEP  K - 1 times
//   PCG_END   last step's chi2; step 4
// K = 3 and 5: 14 launches instead of the 30 of two launches per step.  Small meshes are bound by launches and latency
// (96 x 80 x 3: 174 us -> 95 us), large ones by memory: a step moves 6 vectors instead of 10 (1024^2 x 3: 1568 us ->
// 805 us; 2048^2 x 3: 12.0 ms -> 4.1 ms).
// ------------------------------------------------------------------------------------------
enum { PCG_MASS, PCG_STEP, PCG_G, PCG_M, PCG_END };

// One launch's vectors.  x, r, p: iterate before this launch's step, its residual, the direction before it (x and p
// null: the solve's first step); xo, ro, po: iterate, new residual and direction (PCG_G, PCG_M: ro the next solve's
// right-hand side).  xo must not be x where a neighbour still reads x (PCG_G, PCG_M); r, p and ro, po are different
// vectors.
struct PcgVecs {
    const zd *x, *r, *p;
    zd *xo, *ro, *po;
};

// Partials of a region b: g[b] = <r, r>, g[nreg + b] = <r, OP r>; at a system's first region also its <r, r> and alpha
// of the step before, g[2 nreg + b] and g[3 nreg + b].
template <int NP, int NW, int KIND, bool isM>
__global__ __launch_bounds__(64 * NW) void k_pcg2d(const Sys* sys, const CTile* tiles, const int* mask, const PcgVecs a,
                                                  const zd* v, zd* z, long long NT, const double* gin, double* gout,
                                                  int nreg) {
    using T = double;
    using Row = RowStencil<T>::Row;
    constexpr int IX = kTX - 2 * kPcgHalo, IY = NP * NW - 2 * kPcgHalo;
    __shared__ zd edges[2][NW][2][kTX];
    __shared__ double sums[2], part[NW][2];
    const CTile tile = tiles[blockIdx.x];
    if (mask && !mask[tile.sys]) return;
    const Sys& s = sys[tile.sys];
    const int nx = s.nx, ny = s.ny, lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
    const int ix = lane - kPcgHalo, r0 = wv * NP - kPcgHalo;
    const RegionRows rows0{s.off, (long long)wrapi(tile.x0 + ix, nx), wrapi(tile.y0 + r0, ny), nx, ny};
    const bool own_x = ix >= 0 && ix < IX && tile.x0 + ix < nx;
    auto owned = [&](int i) { return own_x && r0 + i >= 0 && r0 + i < IY && tile.y0 + r0 + i < ny; };
    auto load = [&](const zd* src, zd (&u)[NP]) {
        RegionRows g = rows0;
#pragma unroll
        for (int i = 0; i < NP; ++i, g.next()) u[i] = src[g.at()];
    };
    auto load_owned = [&](const zd* src, zd (&u)[NP]) {
        RegionRows g = rows0;
#pragma unroll
        for (int i = 0; i < NP; ++i, g.next()) u[i] = owned(i) ? src[g.at()] : zd{0.0, 0.0};
    };
    auto store = [&](zd* dst, const zd (&u)[NP]) {
        RegionRows g = rows0;
#pragma unroll
        for (int i = 0; i < NP; ++i, g.next())
            if (owned(i)) dst[g.at()] = u[i];
    };
    zd R[NP], P[NP], X[NP];
    double alpha = 0.0, rho = 0.0;
    if (KIND != PCG_MASS && a.r) {
        load(a.r, R);
        if (a.p) load(a.p, P);
        if (a.x) {
            if constexpr (KIND == PCG_STEP || KIND == PCG_END) load_owned(a.x, X);   // xo may be x
            else load(a.x, X);
        }
        // the sums over the system: its regions' partials in a fixed order (tile.z = its first region)
        const double* g = gin + tile.z;
        const double rho_old = a.p ? g[2LL * nreg] : 0.0, alpha_old = a.p ? g[3LL * nreg] : 0.0;
        const int n = ((nx + IX - 1) / IX) * ((ny + IY - 1) / IY);
        if (wv < 2) {
            double t = 0.0;
            for (int i = lane; i < n; i += 64) t += g[(long long)wv * nreg + i];
            t = wave_sum(t);
            if (lane == 0) sums[wv] = t;
        }
        __syncthreads();
        // D: of the operator that the step's solve belongs to
        const double D = isM ? s.diagM : s.diagL, iD = 1.0 / D;
        rho = sums[0];
        const double beta = rho_old != 0.0 ? rho / rho_old : 0.0;
        const double ia = rho != 0.0 ? sums[1] / (D * rho) - (alpha_old != 0.0 ? beta / alpha_old : 0.0) : 0.0;
        alpha = ia != 0.0 ? 1.0 / ia : 0.0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            P[i] = a.p ? iD * R[i] + beta * P[i] : iD * R[i];
            X[i] = a.x ? X[i] + alpha * P[i] : alpha * P[i];
        }
    } else if constexpr (KIND == PCG_G) {
        load(a.x, X);   // the separable mass inverse has formed x1
    }
    if constexpr (KIND == PCG_END) {
        const T isd = s.isq_dt, isk = s.isq_kap;
        RegionRows g = rows0;
#pragma unroll
        for (int i = 0; i < NP; ++i, g.next())
            if (owned(i)) {
                const long long gi = g.at();
                z[gi] = z[gi] - isk * (z[NT + gi] - isd * X[i]);   // x1 and x2 wait in z
                z[NT + gi] = X[i];
            }
        return;
    }
    const RowStencil<T> op(s);
    auto make = [&](zd l, zd c, zd r) { return op.row(l, c, r); };
    // out(i, OP u, u) at every row, OP = M (mass) or L
    auto apply = [&](auto mass, zd (*edge)[2][kTX], zd (&u)[NP], auto&& out) {
        row_sweep<T, NP, NW>(u, edge, wv, make, [&](int i, const Row& A, const Row& B, const Row& C, zd uB) {
            out(i, decltype(mass)::value ? op.M(A, B, C) : op.L(A, B, C), uB);
        });
    };
    if constexpr (KIND == PCG_MASS) {
        load(v, R);
    } else {
        store(a.xo, X);
        if constexpr (KIND == PCG_STEP) {
            store(a.po, P);
            apply(std::bool_constant<isM>{}, edges[0], P, [&](int i, zd q, zd) { R[i] = R[i] - alpha * q; });
        } else if constexpr (KIND == PCG_G) {
            load(v + NT, R);
            const T k0 = s.kv[0], k1 = s.kv[1], kap = s.kappa;
            row_sweep<T, NP, NW>(X, edges[0], wv, make, [&](int i, const Row& A, const Row& B, const Row& C, zd) {
                R[i] = R[i] - kap * gop(op.K(A, B, C), op.Tj(A, B, C, k0, k1));
            });
        } else {
            apply(std::true_type{}, edges[0], X, [&](int i, zd q, zd) { R[i] = q; });
        }
        store(a.ro, R);
    }
    // the next step's sums
    double acc[2] = {0.0, 0.0};
    apply(std::bool_constant<KIND == PCG_MASS || (KIND == PCG_STEP && isM)>{}, edges[1], R, [&](int i, zd w, zd r) {
        if (!owned(i)) return;
        acc[0] += abs2(r);
        acc[1] += r.x * w.x + r.y * w.y;
    });
    wave_sums<2>(acc, [&](int i, double t) { part[wv][i] = t; });
    __syncthreads();
    if (threadIdx.x < 2) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += part[w][threadIdx.x];
        gout[(long long)threadIdx.x * nreg + blockIdx.x] = t;
    } else if (threadIdx.x == 2 && (int)blockIdx.x == tile.z) {
        gout[2LL * nreg + blockIdx.x] = rho;
        gout[3LL * nreg + blockIdx.x] = alpha;
    }
}

// ------------------------------------------------------------------------------------------
// Meshes of at most 64 x 64 nodes: P^{-1} of a system by one workgroup, CG step by step with its inner products
// over the workgroup.  The order of every sum and the arithmetic per node are those of k_cg_* with 16-row tiles
// (tile q = waves 4 q .. 4 q + 3, a thread's rows four apart), so both give the same bits: with restarts of 30
// and FP32 storage, or residual estimates near rounding, the last digits of the inner solves decide on the
// number of iterations.  The stencils take four consecutive rows per thread (6 rows of x passes for 4 rows of
// results) from p in LDS and hand the result over through LDS; the vectors stay in registers.  Bound by one
// CU's LDS reads and FP64 arithmetic and four barriers per CG step; 64^2 x 3, 3 + 5 + 5 steps: one launch of
// 62 us for 30 of ~4.3 us.
// ------------------------------------------------------------------------------------------
constexpr int kSmallThreads = 1024, kSmallRows = 4;

// v / D correctly rounded, from y = 1 / D correctly rounded (Markstein's two-step division)
__device__ __forceinline__ double div_by(double v, double D, double y) {
    const double q = v * y;
    return __builtin_fma(__builtin_fma(-q, D, v), y, q);
}

// a value equal in every lane, moved to scalar registers (the kernel below is short of vector registers)
__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uniform(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL)), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <typename T>
__global__ __launch_bounds__(kSmallThreads) void k_pcg_small(const Sys* sys, const int* mask, const cx<T>* v, cx<T>* x1,
                                                            cx<T>* x2, cx<T>* z, int mass_iters, int diff_iters,
                                                            int sep, long long NT) {
    __shared__ cx<T> in[kTX * kTX], out[kTX * kTX];
    __shared__ double sums[2][kSmallThreads / 64];
    const int si = blockIdx.x;
    if (mask && !mask[si]) return;
    const Sys& s = sys[si];
    const int nx = s.nx, ny = s.ny, x = (int)threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int yb = (wv >> 2) * 16 + (wv & 3);
    const double diagM = s.diagM, diagL = s.diagL, idM = uniform(1.0 / diagM), idL = uniform(1.0 / diagL);
    auto valid = [&](int i) { return x < nx && yb + 4 * i < ny; };
    auto node = [&](int i) { return s.off + (long long)(yb + 4 * i) * nx + x; };
    auto local = [&](int i) { return (yb + 4 * i) * kTX + x; };
    // of lanes beyond the mesh too (their results are not used): columns of the mesh
    const int xl = x == 0 || x >= nx ? nx - 1 : x - 1, xr = x >= nx - 1 ? 0 : x + 1;
    // u <- f(M u, K u, T u) (K, T: only with WK, WT), u given at the thread's rows
    auto apply = [&](auto wk, auto wt, cx<T> (&u)[kSmallRows], auto&& f) {
        constexpr bool WK = decltype(wk)::value, WT = decltype(wt)::value;
        const T h = T(s.h), m0 = uniform(h * T(1.0 / 6.0)), m1 = uniform(h * T(4.0 / 6.0)), ih = uniform(T(1) / h);
        const T k0 = T(s.kv[0]), k1 = T(s.kv[1]), half = T(0.5);
        auto mass1 = [&](cx<T> l, cx<T> c, cx<T> r) { return m0 * (l + r) + m1 * c; };
        auto diff2 = [&](cx<T> l, cx<T> c, cx<T> r) { return (c + c) - (l + r); };
        auto der1 = [&](cx<T> l, cx<T> r) { return half * (r - l); };
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) in[local(i)] = u[i];
        __syncthreads();
        const int y0 = 4 * wv;
        if (y0 < ny) {
            cx<T> mx[3], kx[3], dx[3];
#pragma unroll
            for (int a = 0; a < kSmallRows + 2; ++a) {
                int y = y0 - 1 + a;
                y = y < 0 ? ny - 1 : y >= ny ? y - ny : y;
                const cx<T>* row = in + y * kTX;
                const cx<T> l = row[xl], c = row[x], r = row[xr];
                mx[2] = mass1(l, c, r);
                if (WK) kx[2] = diff2(l, c, r);   // scaled by ih where it is used, where it rounds as in stencil()
                if (WT) dx[2] = der1(l, r);
                if (a >= 2) {
                    const cx<T> Mu = mass1(mx[0], mx[1], mx[2]);
                    cx<T> Ku{T(0), T(0)}, Tu{T(0), T(0)};
                    if (WK) {
                        // mass1 of ih kx, contracted as the compiler does where all rows are in one block
                        const cx<T> k2 = ih * kx[2];
                        const cx<T> ks{mad(ih, kx[0].x, k2.x), mad(ih, kx[0].y, k2.y)};
                        Ku = (m0 * ks + m1 * (ih * kx[1])) + ih * diff2(mx[0], mx[1], mx[2]);
                    }
                    if (WT) Tu = T(2) * (k0 * mass1(dx[0], dx[1], dx[2]) + k1 * der1(mx[0], mx[2]));
                    if (x < nx && y0 + a - 2 < ny) out[(y0 + a - 2) * kTX + x] = f(Mu, Ku, Tu);
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    mx[j] = mx[j + 1];
                    if (WK) kx[j] = kx[j + 1];
                    if (WT) dx[j] = dx[j + 1];
                }
                __builtin_amdgcn_sched_barrier(0);   // later rows' loads would hold registers the vectors need
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) u[i] = out[local(i)];
    };
    int set = 0;
    // sum over the system: per tile of four waves, then over the tiles t as (0 + 2) + (1 + 3); two sets of wave
    // totals in turn, so one barrier
    auto total = [&](double acc) {
        const double w = wave_sum(acc);
        if (x == 0) sums[set][wv] = w;
        __syncthreads();
        double t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double* l = sums[set] + 4 * q;
            t[q] = ((l[0] + l[1]) + l[2]) + l[3];
        }
        set ^= 1;
        return uniform((t[0] + t[2]) + (t[1] + t[3]));
    };
    auto norm2 = [](double a, double b) { return mad(a, a, b * b); };
    // n CG steps on OP (0: M, 1: L) from zero for the residual r; p = r / D and rho = r^H r / D given
    auto solve = [&](auto opc, int n, double rho, cx<T> (&r)[kSmallRows], cx<T> (&p)[kSmallRows],
                     cx<T> (&xv)[kSmallRows]) {
        constexpr int OP = decltype(opc)::value;
        const double D = OP == 0 ? diagM : diagL, y = OP == 0 ? idM : idL;
        const T iD = T(y);
        const T cM = OP == 0 ? T(1) : T(s.isq_dt), cK = OP == 0 ? T(0) : T(s.sq_kap);
        T beta = T(0);
        for (int it = 0; it < n; ++it) {
            if (it > 0)
#pragma unroll
                for (int i = 0; i < kSmallRows; ++i)
                    if (valid(i)) p[i] = iD * r[i] + beta * p[i];
            cx<T> q[kSmallRows];
#pragma unroll
            for (int i = 0; i < kSmallRows; ++i) q[i] = p[i];
            apply(std::integral_constant<bool, OP == 1>{}, std::false_type{}, q,
                  [&](cx<T> Mu, cx<T> Ku, cx<T>) { return OP == 0 ? Mu : cM * Mu + cK * Ku; });
            double acc = 0.0;
#pragma unroll
            for (int i = 0; i < kSmallRows; ++i)
                if (valid(i)) {
                    const cx<T> pc = p[i], qv = q[i];
                    acc += double(pc.x) * double(qv.x) + double(pc.y) * double(qv.y);
                }
            const double pq = total(acc);
            const T alpha = uniform((rho != 0.0 && pq != 0.0) ? T(rho / pq) : T(0));
            const bool last = it == n - 1;
            acc = 0.0;
#pragma unroll
            for (int i = 0; i < kSmallRows; ++i)
                if (valid(i)) {
                    if (it == 0)
                        xv[i] = alpha * p[i];
                    else
                        xv[i] = xv[i] + alpha * p[i];
                    if (!last) {
                        const cx<T> rv = r[i] - alpha * q[i];
                        r[i] = rv;
                        acc += div_by(norm2(rv.x, rv.y), D, y);
                    }
                }
            if (last) break;
            const double rho1 = total(acc);
            beta = uniform(rho != 0.0 ? T(rho1 / rho) : T(0));
            rho = rho1;
        }
    };
    cx<T> r[kSmallRows], p[kSmallRows], xv[kSmallRows];
    // step 1: x1 ~ M^{-1} beta1
    if (sep) {
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) xv[i] = x1[node(i)];
    } else {
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) {
                const cx<T> rv = v[node(i)];
                r[i] = rv;
                p[i] = T(idM) * rv;
                acc += norm2(rv.x, rv.y) * idM;
            }
        solve(std::integral_constant<int, 0>{}, mass_iters, total(acc), r, p, xv);
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) x1[node(i)] = xv[i];
    }
    // step 2: x2 ~ L^{-1} (beta2 - kappa G x1)
    {
        apply(std::true_type{}, std::true_type{}, xv, [&](cx<T>, cx<T> Ku, cx<T> Tu) { return gop(Ku, Tu); });
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) {
                const cx<T> rv = v[NT + node(i)] - T(s.kappa) * xv[i];
                r[i] = rv;
                p[i] = T(idL) * rv;
                acc += div_by(norm2(rv.y, rv.x), diagL, idL);   // this order, as k_cg_init_g contracts it
            }
        solve(std::integral_constant<int, 1>{}, diff_iters, total(acc), r, p, xv);
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) x2[node(i)] = xv[i];
    }
    // steps 3 and 4: chi2 ~ L^{-1} M x2, chi1
    {
        apply(std::false_type{}, std::false_type{}, xv, [&](cx<T> Mu, cx<T>, cx<T>) { return Mu; });
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) {
                r[i] = xv[i];
                p[i] = T(idL) * xv[i];
                acc += div_by(norm2(xv[i].x, xv[i].y), diagL, idL);
            }
        solve(std::integral_constant<int, 1>{}, diff_iters, total(acc), r, p, xv);
        const T isd = T(s.isq_dt), isk = T(s.isq_kap);
#pragma unroll
        for (int i = 0; i < kSmallRows; ++i)
            if (valid(i)) {
                const long long gi = node(i);
                z[NT + gi] = xv[i];
                z[gi] = x1[gi] - isk * (x2[gi] - isd * xv[i]);
            }
    }
}

template <typename T>
void launch_precond_pcg_small(const Dev& d, const cx<T>* v, cx<T>* z, cx<T>* x1, cx<T>* x2, int mass_iters,
                              int diff_iters, int mass_sep, const int* mask, hipStream_t st) {
    if (mass_sep > 0) launch_mass_sep<T>(d, mass_sep, v, x1, mask, st);
    ProbeScope ps(d, KID_PCG_SPMV, st, (double)d.NT * sizeof(cx<T>) * 4.0, mask, true);
    ps.launch(k_pcg_small<T>, dim3(d.S), dim3(kSmallThreads), d.sys, mask, v, x1, x2, z, mass_iters, diff_iters,
              mass_sep, d.NT);
}
template void launch_precond_pcg_small<double>(const Dev&, const zd*, zd*, zd*, zd*, int, int, int, const int*,
                                               hipStream_t);
template void launch_precond_pcg_small<float>(const Dev&, const zf*, zf*, zf*, zf*, int, int, int, const int*,
                                              hipStream_t);

template <int NP, int NW>
static void pcg_launches(const Dev& d, const CTile* tiles, int nreg, const zd* v, zd* z, zd* const* w, double* part,
                         int mass_iters, int diff_iters, int mass_sep, const int* mask, hipStream_t st) {
    using std::integral_constant;
    const double vec = (double)d.NT * sizeof(zd);
    double* G[2] = {part, part + (long long)kPcgSums * nreg};
    zd *x = w[0], *R[2] = {w[1], w[2]}, *P[2] = {w[3], w[4]};
    PcgVecs a{};
    int g = 0;
    auto go = [&](auto kind, auto mass, double vecs) {
        ProbeScope ps(d, KID_PCG_SPMV, st, vec * vecs, mask, true);
        ps.launch(k_pcg2d<NP, NW, decltype(kind)::value, decltype(mass)::value>, dim3(nreg), dim3(64 * NW), d.sys,
                  tiles, mask, a, v, z, d.NT, G[g], G[g ^ 1], nreg);
        g ^= 1;
    };
    // steps 1 .. n - 1 of a solve for the right-hand side r, whose sums the launch before has left
    auto steps = [&](auto mass, int n, const zd* r) {
        a = PcgVecs{nullptr, r, nullptr, x, nullptr, nullptr};
        int b = r == R[0] ? 1 : 0;
        for (int k = 1; k < n; ++k, b ^= 1) {
            a.ro = R[b];
            a.po = P[b];
            go(integral_constant<int, PCG_STEP>{}, mass, a.p ? 6.0 : 4.0);
            a = PcgVecs{x, a.ro, a.po, x, nullptr, nullptr};
        }
    };
    // where the next solve's right-hand side goes
    auto next = [&](zd* xo) {
        a.xo = xo;
        return a.ro = a.r == R[0] ? R[1] : R[0];
    };
    const zd* r;
    if (mass_sep > 0) {
        launch_mass_sep<double>(d, mass_sep, v, x, mask, st);
        a.x = x;
        r = next(z);
        go(integral_constant<int, PCG_G>{}, std::true_type{}, 4.0);
    } else {
        go(integral_constant<int, PCG_MASS>{}, std::true_type{}, 1.0);
        steps(std::true_type{}, mass_iters, v);
        r = next(z);
        go(integral_constant<int, PCG_G>{}, std::true_type{}, a.p ? 6.0 : 4.0);
    }
    steps(std::false_type{}, diff_iters, r);
    r = next(z + d.NT);
    go(integral_constant<int, PCG_M>{}, std::false_type{}, a.p ? 5.0 : 3.0);
    steps(std::false_type{}, diff_iters, r);
    go(integral_constant<int, PCG_END>{}, std::false_type{}, a.p ? 7.0 : 5.0);
}

void launch_precond_pcg2d(const Dev& d, int shape, const CTile* tiles, int nreg, const zd* v, zd* z, zd* const* w,
                          double* part, int mass_iters, int diff_iters, int mass_sep, const int* mask, hipStream_t st) {
    auto go = [&](auto i) {
        constexpr int I = decltype(i)::value;
        pcg_launches<kPcgShape[I][0], kPcgShape[I][1]>(d, tiles, nreg, v, z, w, part, mass_iters, diff_iters, mass_sep, mask,
                                                       st);
    };
    static_assert(sizeof(kPcgShape) / sizeof(kPcgShape[0]) == 3, "one case per shape");
    if (shape == 0) go(std::integral_constant<int, 0>{});
    else if (shape == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 2>{});
}

}  // namespace apfc
