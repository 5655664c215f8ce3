// The block preconditioner of Eq. (12) with Jacobi-PCG inner solves, fused per step on register-resident
// regions (2D), for gfx950, with its launcher.
#include "kernels_region.h"

namespace apfc {

// ------------------------------------------------------------------------------------------
// K steps of Jacobi-PCG from a zero start on OP (constant diagonal D) give the vector of the Krylov space
// span{b, OP b, .., OP^{K-1} b} with the smallest OP-norm error, so the two inner products per step need not
// be taken one after the other: with t_i = T_i(A) b, A = (D^{-1} OP - theta) / delta the operator mapped to
// [-1, 1] (exact symbol bounds theta -+ delta) and T_i the Chebyshev polynomials, the result is
//   x = sum_{i < K} c_i t_i,   H c = g,   H_ij = <t_i, OP t_j>,   g_i = <t_i, b>,
// and A t_j = (t_{j-1} + t_{j+1}) / 2 (t_1 for j = 0) gives H from the Gram matrix of t_0 .. t_K.  A solve is
// then two halves without a global reduction inside: the Gram matrix of its right-hand side (partials per
// region), and, in the next launch, the K x K system and the sum over the t_i, formed again from b.  The
// Chebyshev basis keeps H well conditioned; a direction whose pivot is lost to rounding (b in a smaller
// invariant space, where CG has converged already) is left out together with the later ones.
//
// A workgroup holds a region of 64 x 8 NP nodes = interior + `halo` layers in registers (reg_sweep; one wave
// per NP rows), each stencil application exact one layer further in.  Launches per application of P^{-1}:
//   STAGE 0: Gram matrix of beta1                              (mass solve)
//   STAGE 1: x1 from it; r2 = beta2 - kappa G x1, its Gram matrix (SEP: x1 given)
//   STAGE 2: x2 from it; r3 = M x2, its Gram matrix
//   STAGE 3: chi2 from it; step 4
// Latency bounds them at the sizes they are used for (108 regions on 256^2 x 3: one per CU): four launches of
// 11 + 35 + 35 + 15 us stand for the 30 launches (~150 us) that one launch per CG half-step takes.
// ------------------------------------------------------------------------------------------

// Gram pair (i, j), i <= j, of t_0 .. t_K as slot j (j + 1) / 2 + i
__host__ __device__ constexpr int gram_slot(int i, int j) { return j * (j + 1) / 2 + i; }

// The K coefficients c of one solve from the Gram matrix G (slots; pair (K, K) not needed), for the operator
// with diagonal D and scaled spectrum theta -+ delta.  One thread.
__device__ void krylov_coef(const double* G, int K, double D, double theta, double delta, double* c) {
    constexpr int KM = kPcgMax;
    const double tol = 1e-14;   // pivots below tol H_00 are rounding
    double L[KM][KM], d[KM], y[KM];
    auto g = [&](int i, int j) { return i <= j ? G[gram_slot(i, j)] : G[gram_slot(j, i)]; };
    auto at = [&](int i, int j) { return j == 0 ? g(i, 1) : 0.5 * (g(i, j - 1) + g(i, j + 1)); };
    int n = 0;
    bool more = true;
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        c[j] = 0.0;
        if (j >= K || !more) continue;
        // row j of H (i <= j) and the pivot; L row-wise
        double row[KM];
#pragma unroll
        for (int i = 0; i <= j; ++i) {
            double h = theta * g(i, j) + 0.5 * delta * (at(i, j) + at(j, i));
#pragma unroll
            for (int q = 0; q < i; ++q) h -= L[i][q] * row[q];
            row[i] = h;                                  // L_ji d_i (i < j), d_j (i = j)
        }
        double piv = theta * g(j, j) + delta * at(j, j);
        double yv = g(0, j);
#pragma unroll
        for (int q = 0; q < j; ++q) {
            const double l = row[q] * d[q];              // d holds the inverse pivots
            piv -= l * row[q];
            L[j][q] = l;
            yv -= l * y[q];
        }
        if (!(piv > tol * (theta * g(0, 0) + delta * g(0, 1)))) {
            more = false;
            continue;
        }
        d[j] = 1.0 / piv;
        y[j] = yv;
        n = j + 1;
    }
#pragma unroll
    for (int i = KM - 1; i >= 0; --i) {
        if (i >= n) continue;
        double v = y[i] * d[i];
#pragma unroll
        for (int q = i + 1; q < KM; ++q)
            if (q < n) v -= L[q][i] * c[q];
        c[i] = v;
    }
#pragma unroll
    for (int i = 0; i < KM; ++i) c[i] = i < n ? c[i] / D : 0.0;
}

// OP mapped to [-1, 1] in split form: A u = a (pA + pC) + b pB + c (uA + uC) + d uB
struct MappedOp {
    double a, b, c, d;
};
__device__ __forceinline__ MappedOp mapped_op(const Sys& s, bool isM) {
    const SplitCoef o = split_coef(s.h, isM ? 1.0 : s.isq_dt, isM ? 0.0 : s.sq_kap);
    const double th = isM ? s.thM : s.thL, de = isM ? s.deM : s.deL, D = isM ? s.diagM : s.diagL;
    const double f = 1.0 / (D * de);
    return {f * o.a, f * o.b, f * o.c, f * o.d - th / de};
}

template <int NP, int STAGE, bool SEP>
__global__ __launch_bounds__(kPcgThreads, 2) void k_pcg2d(const Sys* sys, const CTile* tiles, const int* mask,
                                                         const zd* v, zd* x1, zd* x2, zd* r2, zd* r3, zd* z, int KM1,
                                                         int KL, int halo, long long NT, const double* gin,
                                                         double* gout, int nreg) {
    using T = double;
    constexpr int KM = kPcgMax, NW = kPcgThreads / 64, RX = kTX, RY = NP * NW;
    constexpr bool SOLVE = STAGE >= 1 && !(STAGE == 1 && SEP), GRAM = STAGE <= 2;
    __shared__ zd edges[2][NW][2][kTX];
    __shared__ double sums[kPcgGram], coef[KM], part[GRAM ? NW : 1][kPcgGram];
    const CTile tile = tiles[blockIdx.x];
    if (mask && !mask[tile.sys]) return;
    const Sys& s = sys[tile.sys];
    const int nx = s.nx, ny = s.ny, lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
    const int IX = RX - 2 * halo, IY = RY - 2 * halo, r0 = wv * NP;
    const RegionRows rows0{s.off, (long long)wrapi(tile.x0 - halo + lane, nx), wrapi(tile.y0 - halo + r0, ny), nx, ny};
    const int ix = lane - halo;
    const bool own_x = ix >= 0 && ix < IX && tile.x0 + ix < nx;
    auto owned = [&](int i) {
        const int iy = r0 + i - halo;
        return own_x && iy >= 0 && iy < IY && tile.y0 + iy < ny;
    };
    auto load = [&](const zd* src, zd (&u)[NP]) {
        RegionRows g = rows0;
#pragma unroll
        for (int i = 0; i < NP; ++i, g.next()) u[i] = src[g.at()];
    };
    auto store = [&](zd* dst, const zd (&u)[NP]) {
        RegionRows g = rows0;
#pragma unroll
        for (int i = 0; i < NP; ++i, g.next())
            if (owned(i)) dst[g.at()] = u[i];
    };
    int e = 0;   // edge set of the next sweep (two sets in turn: one barrier per sweep)
    // t_{i+1} (out) = f A t_i - (i > 0 ? t_{i-1} : 0), f = 1 for i = 0 and 2 after it
    auto advance = [&](const MappedOp& o, bool isM, T f, zd (&t)[NP], auto&& out) {
        const T a = f * T(o.a), b = f * T(o.b), cc = f * T(o.c), dd = f * T(o.d);
        reg_sweep<T, NP, NW, false>(t, edges[e], wv, [&](int i, zd pA, zd pB, zd pC, zd uA, zd uB,
                                                         zd uC, zd, zd, zd) {
            zd q = a * (pA + pC) + b * pB + dd * uB;
            if (!isM) q = q + cc * (uA + uC);
            out(i, uB, q);
        });
        e ^= 1;
    };
    zd r[NP];   // the right-hand side whose Gram matrix this stage forms
    if constexpr (SOLVE) {
        constexpr bool isM = STAGE == 1;
        const int K = isM ? KM1 : KL;
        zd U[NP], P[NP], X[NP];
        load(STAGE == 1 ? v : STAGE == 2 ? r2 : r3, U);
        // the system's Gram matrix: its regions' partials in a fixed order (tile.z = its first region)
        {
            const int n = ((nx + IX - 1) / IX) * ((ny + IY - 1) / IY);
            for (int q = wv; q < gram_slot(K, K); q += NW) {
                double a = 0.0;
                for (int t = lane; t < n; t += 64) a += gin[(long long)q * nreg + tile.z + t];
                a = wave_sum(a);
                if (lane == 0) sums[q] = a;
            }
            __syncthreads();
            if (threadIdx.x == 0)
                krylov_coef(sums, K, isM ? s.diagM : s.diagL, isM ? s.thM : s.thL, isM ? s.deM : s.deL, coef);
            __syncthreads();
        }
        const MappedOp o = mapped_op(s, isM);
        const T c0 = T(coef[0]);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            X[i] = c0 * U[i];
            P[i] = zd{T(0), T(0)};
        }
        for (int k = 1; k < K; ++k) {
            const T c = T(coef[k]);
            advance(o, isM, k == 1 ? T(1) : T(2), U, [&](int i, zd tk, zd q) {
                const zd tn = q - P[i];
                P[i] = tk;
                U[i] = tn;
                X[i] = X[i] + c * tn;
            });
        }
        if constexpr (STAGE == 3) {
            const T isd = T(s.isq_dt), isk = T(s.isq_kap);
            RegionRows g = rows0;
#pragma unroll
            for (int i = 0; i < NP; ++i, g.next())
                if (owned(i)) {
                    const long long gi = g.at();
                    z[gi] = x1[gi] - isk * (x2[gi] - isd * X[i]);
                    z[NT + gi] = X[i];
                }
            return;
        }
        store(STAGE == 1 ? x1 : x2, X);
#pragma unroll
        for (int i = 0; i < NP; ++i) U[i] = X[i];
        if constexpr (STAGE == 1) {
            load(v + NT, r);
        }
        const T k3 = T(s.kappa / 3.0), k4 = T(4.0 * s.kappa), kap = T(s.kappa);
        const T g0 = T(s.kappa * s.h / 6.0 * s.kv[0]), g1 = T(s.kappa * s.h / 6.0 * s.kv[1]);
        const SplitCoef m = split_coef(s.h, 1.0, 0.0);
        const T ma = T(m.a), mb = T(m.b);
        reg_sweep<T, NP, NW, STAGE == 1>(U, edges[e], wv, [&](int i, zd pA, zd pB, zd pC, zd uA, zd uB,
                                                              zd uC, zd eA, zd eB, zd eC) {
            if constexpr (STAGE == 1) {
                const zd kk = kap * (uA + uC) + k4 * uB - k3 * ((pA + pC) + pB);
                const zd tt = g0 * (T(4) * eB + (eA + eC)) + g1 * (pC - pA);
                r[i] = r[i] + zd{kk.x + tt.y, kk.y - tt.x};
            } else {
                r[i] = ma * (pA + pC) + mb * pB;
            }
        });
        e ^= 1;
        store(STAGE == 1 ? r2 : r3, r);
    } else if constexpr (STAGE == 0) {
        load(v, r);
    } else {
        // the separable mass inverse has formed x1
        zd U[NP];
        load(x1, U);
        load(v + NT, r);
        const T k3 = T(s.kappa / 3.0), k4 = T(4.0 * s.kappa), kap = T(s.kappa);
        const T g0 = T(s.kappa * s.h / 6.0 * s.kv[0]), g1 = T(s.kappa * s.h / 6.0 * s.kv[1]);
        reg_sweep<T, NP, NW, true>(U, edges[e], wv, [&](int i, zd pA, zd pB, zd pC, zd uA, zd uB,
                                                        zd uC, zd eA, zd eB, zd eC) {
            const zd kk = kap * (uA + uC) + k4 * uB - k3 * ((pA + pC) + pB);
            const zd tt = g0 * (T(4) * eB + (eA + eC)) + g1 * (pC - pA);
            r[i] = r[i] + zd{kk.x + tt.y, kk.y - tt.x};
        });
        e ^= 1;
        store(r2, r);
    }
    if constexpr (GRAM) {
        constexpr bool isM = STAGE == 0;
        const int K = isM ? KM1 : KL;
        const MappedOp o = mapped_op(s, isM);
        zd t[KM + 1][NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) t[0][i] = r[i];
#pragma unroll
        for (int j = 0; j <= KM; ++j) {
            if (j > K) continue;
            if (j > 0)
                advance(o, isM, j == 1 ? T(1) : T(2), t[j > 0 ? j - 1 : 0], [&](int i, zd, zd q) {
                    t[j][i] = j > 1 ? q - t[j > 1 ? j - 2 : 0][i] : q;
                });
            double acc[KM + 1];
#pragma unroll
            for (int q = 0; q <= j; ++q) acc[q] = 0.0;
#pragma unroll
            for (int i = 0; i < NP; ++i)
                if (owned(i)) {
                    const double re = t[j][i].x, im = t[j][i].y;
#pragma unroll
                    for (int q = 0; q <= j; ++q) acc[q] += double(t[q][i].x) * re + double(t[q][i].y) * im;
                }
#pragma unroll
            for (int q = 0; q <= j; ++q)
                if (gram_slot(q, j) < kPcgGram) {   // pair (KM, KM) is not needed
                    const double w = wave_sum(acc[q]);
                    if (lane == 0) part[wv][gram_slot(q, j)] = w;
                }
        }
        __syncthreads();
        if ((int)threadIdx.x < gram_slot(K, K)) {
            double a = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) a += part[w][threadIdx.x];
            gout[(long long)threadIdx.x * nreg + blockIdx.x] = a;
        }
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
    const int xl = x == 0 ? nx - 1 : x - 1, xr = x == nx - 1 ? 0 : x + 1;
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

// Halo of the fused regions: stage 1 forms x1 (mass_iters - 1 layers), G x1 and diff_iters layers of t_i;
// stage 2 x2, M x2 and the t_i.
int pcg_halo(int mass_iters, int diff_iters, bool sep) {
    const int s1 = (sep ? 0 : mass_iters - 1) + 1 + diff_iters, s2 = 2 * diff_iters;
    return s1 > s2 ? s1 : s2;
}

template <int NP>
static void pcg_stages(const Dev& d, const CTile* tiles, int nreg, const zd* v, zd* z, zd* x1, zd* x2, zd* r2, zd* r3,
                       double* gram, int mass_iters, int diff_iters, int mass_sep, const int* mask, hipStream_t st) {
    const int halo = pcg_halo(mass_iters, diff_iters, mass_sep > 0);
    const dim3 g(nreg), b(kPcgThreads);
    double* G[2] = {gram, gram + (long long)kPcgGram * nreg};
    const double vec = (double)d.NT * sizeof(zd);
    auto go = [&](auto stage, auto sep, double vecs, const double* gin, double* gout) {
        ProbeScope ps(d, KID_PCG_SPMV, st, vec * vecs, mask, true);
        ps.launch(k_pcg2d<NP, decltype(stage)::value, decltype(sep)::value>, g, b, d.sys, tiles, mask, v, x1, x2,
                  r2, r3, z, mass_iters, diff_iters, halo, d.NT, gin, gout, nreg);
    };
    using std::integral_constant;
    if (mass_sep > 0) {
        launch_mass_sep<double>(d, mass_sep, v, x1, mask, st);
        go(integral_constant<int, 1>{}, std::true_type{}, 3.0, nullptr, G[1]);
    } else {
        go(integral_constant<int, 0>{}, std::false_type{}, 1.0, nullptr, G[0]);
        go(integral_constant<int, 1>{}, std::false_type{}, 4.0, G[0], G[1]);
    }
    go(integral_constant<int, 2>{}, std::false_type{}, 3.0, G[1], G[0]);
    go(integral_constant<int, 3>{}, std::false_type{}, 5.0, G[0], nullptr);
}

void launch_precond_pcg2d(const Dev& d, int rows, const CTile* tiles, int nreg, const zd* v, zd* z, zd* x1, zd* x2,
                          zd* r2, zd* r3, double* gram, int mass_iters, int diff_iters, int mass_sep, const int* mask,
                          hipStream_t st) {
    if (rows == kPcgRows[0])
        pcg_stages<kPcgRows[0]>(d, tiles, nreg, v, z, x1, x2, r2, r3, gram, mass_iters, diff_iters, mass_sep, mask, st);
    else
        pcg_stages<kPcgRows[1]>(d, tiles, nreg, v, z, x1, x2, r2, r3, gram, mass_iters, diff_iters, mass_sep, mask, st);
}

}  // namespace apfc
