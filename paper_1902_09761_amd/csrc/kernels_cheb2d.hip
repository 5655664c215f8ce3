// The block preconditioner of Eq. (12) with Chebyshev-Jacobi inner solves, fused per step on LDS regions
// (2D), for gfx950, with its launcher.
#include "kernels_region.h"

namespace apfc {

// ------------------------------------------------------------------------------------------
// Block preconditioner with Chebyshev-Jacobi inner solves, fused per step (2D).
//
// A workgroup owns a region of RX x RY nodes = an interior tile plus `halo` layers (periodic wrap).
// Every stencil application inside the region is evaluated from the region's values (staged in LDS, or,
// for FP32 regions one wave wide, held in registers with the edge rows of the waves exchanged through
// LDS) and is exact one layer further in than the previous one, so after `halo` applications the interior
// holds the same values an unfused sweep over the whole mesh would give.  Stages 0 and 1 can also form
// their half of the next FGMRES basis vector as they load it (VIn).  Three kernels per preconditioner
// application:
//   STAGE 0: x1   = Cheb_M^{sM}(beta1)                         (step 1)
//   STAGE 1: x2   = Cheb_L^{sL}(beta2 - kappa G x1)             (step 2)
//   STAGE 2: chi2 = Cheb_L^{sL}(M x2);  chi1 = x1 - (x2 - chi2/sqrt(dt))/sqrt(kappa)   (steps 3, 4)
// Chebyshev iteration for D^{-1} A with spectrum in [theta - delta, theta + delta], x0 = 0
// (three-term recurrence on the correction d):
//   d0 = r0/(theta D), rho0 = delta/theta; x_{k+1} = x_k + d_k;
//   r_{k+1} = r_k - A d_k; rho_{k+1} = 1/(2 theta/delta - rho_k);
//   d_{k+1} = rho_{k+1} rho_k d_k + (2 rho_{k+1}/delta) D^{-1} r_{k+1}.
// The spectral bounds are exact for the constant-coefficient operators (symbol extremes at the
// corners cos(theta_d) = +-1), so the iteration needs no inner products.
// ------------------------------------------------------------------------------------------
// Operators in split form (kernels_region.h).
// The LDS region keeps one pad row above and below the RY region rows (region row q at LDS row q + 1),
// so a thread's rows r0 - 1 .. r0 + NP are rows of the array with no clamping and every load of the
// sweep is a fixed offset from the thread's three column addresses.  split_sweep streams them (b = LDS row
// r0 of the buffer, i.e. region row r0 - 1; columns xm, xc, xp) and calls
// f(i, pA, pB, pC, uA, uB, uC, eA, eB, eC) for region row r0 + i (e only with WE).  The loads of the next
// row are issued while the current one is used, and no further (a scheduling barrier per row): hoisting
// every row's loads ahead would cost registers the workgroups of a CU need.
template <typename T, int NP, int RX, bool WE, typename F>
__device__ __forceinline__ void split_sweep(const cx<T>* b, int xm, int xc, int xp, F&& f) {
    const cx<T> zero{T(0), T(0)};
    cx<T> pA = zero, pB = zero, uA = zero, uB = zero, eA = zero, eB = zero;
    const cx<T>* bm = b + xm;
    const cx<T>* bc = b + xc;
    const cx<T>* bp = b + xp;
    cx<T> l = bm[0], c = bc[0], r = bp[0];
#pragma unroll
    for (int a = 0; a < NP + 2; ++a) {
        cx<T> ln = zero, cn = zero, rn = zero;
        if (a + 1 < NP + 2) {
            ln = bm[(a + 1) * RX];
            cn = bc[(a + 1) * RX];
            rn = bp[(a + 1) * RX];
        }
        const cx<T> pC = T(4) * c + (l + r);
        const cx<T> eC = WE ? r - l : zero;
        if (a >= 2) f(a - 2, pA, pB, pC, uA, uB, c, eA, eB, eC);
        pA = pB; pB = pC;
        uA = uB; uB = c;
        eA = eB; eB = eC;
        l = ln; c = cn; r = rn;
        __builtin_amdgcn_sched_barrier(0);
    }
}

// FP32 (mixed precision): two region buffers used in turn; iteration k reads the correction d_{k-1} from
// one and writes d_k into the other as soon as it is formed, so each iteration needs one barrier and d_k
// needs no registers (a thread's own d_{k-1} is the centre value of its sweep).  FP64 regions are twice
// as large: one buffer, d_k kept in registers until the sweep has finished reading.
template <typename T>
constexpr int cheb_buffers() { return sizeof(T) == 4 ? 2 : 1; }

// MR > 0 (stage 0 only): x1 = W beta1 with the separable mass inverse of MR taps per side (Sys::wsep; the
// operator of launch_mass_sep) instead of the Chebyshev mass iterations: an x filter of the region's rows,
// then a y filter at the thread's rows.
template <typename T, int STAGE, int RX, int RY, int NTH, int MR = 0>
__global__ __launch_bounds__(NTH, sizeof(T) == 4 ? 4 : 2) void k_cheb2d(
    const Sys* sys, const CTile* tiles, const int* mask, const cx<T>* v, cx<T>* x1, cx<T>* x2, cx<T>* z, int sM,
    int sL, int halo, long long NT, VIn<T> vin) {
    // the separable stage 0 needs one region buffer: half the LDS, twice the workgroups per CU
    constexpr int NB = MR > 0 ? 1 : cheb_buffers<T>();
    constexpr int RL = RY + 2, RP = RX * RL, NP = RX * RY / NTH;
    static_assert((RX * RY) % NTH == 0 && NTH % RX == 0, "region rows must map onto whole workgroup rows");
    // RG: the Chebyshev stages of FP32 regions one wave wide keep the thread's rows in registers
    // (reg_sweep); the region is not staged in LDS, only the edge rows of the waves' blocks (two sets, used
    // in turn by consecutive sweeps, so each sweep needs one barrier)
    constexpr bool RG = MR == 0 && RX == kTX && sizeof(T) == 4;
    constexpr int NW = NTH / RX;
    __shared__ cx<T> bufs[RG ? 1 : NB][RG ? 1 : RP];
    __shared__ cx<T> edges[RG ? 2 : 1][RG ? NW : 1][2][kTX];
    const int wv = (int)threadIdx.x / RX;
    const CTile tile = tiles[blockIdx.x];
    if (mask && !mask[tile.sys]) return;
    const Sys s = sys[tile.sys];
    const int IX = RX - 2 * halo, IY = RY - 2 * halo;
    // thread -> region column px and NP consecutive rows r0 .. r0 + NP - 1
    const int px = threadIdx.x % RX, r0 = (threadIdx.x / RX) * NP;
    const int xm = px > 0 ? px - 1 : px, xp = px < RX - 1 ? px + 1 : px;
    const RegionRows rows0{s.off, (long long)wrapi(tile.x0 - halo + px, s.nx), wrapi(tile.y0 - halo + r0, s.ny), s.nx,
                           s.ny};
    auto lrow = [&](cx<T>* b, int i) -> cx<T>& { return b[(r0 + 1 + i) * RX + px]; };
    // the pad rows only feed the outermost halo rows; zero them so that no stale value is ever read
    if constexpr (!RG)
        for (int e = threadIdx.x; e < RX; e += NTH)
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                bufs[q][e] = cx<T>{T(0), T(0)};
                bufs[q][(RL - 1) * RX + e] = cx<T>{T(0), T(0)};
            }
    cx<T> X[NP], R[NP];
    constexpr int PC = NP % 4 == 0 ? 4 : NP % 3 == 0 ? 3 : NP % 2 == 0 ? 2 : 1;
    // nodes the region owns (its interior; no wrap: each mesh node is owned by exactly one region)
    const int ix = px - halo;
    const bool own_x = ix >= 0 && ix < IX && tile.x0 + ix < s.nx;
    auto own_row = [&](int i) {
        const int iy = r0 + i - halo;
        return iy >= 0 && iy < IY && tile.y0 + iy < s.ny;
    };
    // The input half at offset hoff into R: v, or the basis vector formed from vin (normalised, and projected
    // against the earlier basis vectors, here instead of in a pass of its own), whose owned nodes are also
    // stored to vin.vout
    auto load_in = [&](long long hoff) {
        RegionRows g = rows0;
        if (!vin.src) {
#pragma unroll
            for (int i = 0; i < NP; ++i, g.next()) R[i] = v[hoff + g.at()];
            return;
        }
        const double* hc = vin.hcoef + (long long)tile.sys * vin.hld;
        const double sc = vin.scale[tile.sys];
        // PC rows at a time: FP64 accumulators for all NP rows would cost a third of the workgroups per CU
#pragma unroll
        for (int i0 = 0; i0 < NP; i0 += PC) {
            zd u[PC];
            long long gi[PC];
#pragma unroll
            for (int i = 0; i < PC; ++i, g.next()) {
                gi[i] = hoff + g.at();
                u[i] = ld<double>(vin.src, gi[i]);
            }
            for (int l = 0; l < vin.nv; ++l) {
                const zd c{hc[2 * l], hc[2 * l + 1]};
                const cx<T>* Vl = vin.V + l * vin.vs;
#pragma unroll
                for (int i = 0; i < PC; ++i) u[i] = u[i] - cmul(c, ld<double>(Vl, gi[i]));
            }
#pragma unroll
            for (int i = 0; i < PC; ++i) {
                R[i0 + i] = cx<T>{T(sc * u[i].x), T(sc * u[i].y)};
                if (own_x && own_row(i0 + i)) vin.vout[gi[i]] = R[i0 + i];
            }
        }
    };
    // right-hand side of the inner solve
    if constexpr (STAGE == 0) {
        load_in(0);
    } else {
        // stage 1: r = beta2 - kappa G x1 with G = -K + i T_j (r += kappa K x1 - i kappa T_j x1); stage 2: r = M x2
        const T k3 = T(s.kappa / 3.0), k4 = T(4.0 * s.kappa), kap = T(s.kappa);
        const T g0 = T(s.kappa * s.h / 6.0 * s.kv[0]), g1 = T(s.kappa * s.h / 6.0 * s.kv[1]);
        const SplitCoef m = split_coef(s.h, 1.0, 0.0);
        const T ma = T(m.a), mb = T(m.b);
        auto rhs = [&](int i, cx<T> pA, cx<T> pB, cx<T> pC, cx<T> uA, cx<T> uB, cx<T> uC, cx<T> eA, cx<T> eB,
                       cx<T> eC) {
            if constexpr (STAGE == 1) {
                const cx<T> kk = kap * (uA + uC) + k4 * uB - k3 * ((pA + pC) + pB);
                const cx<T> tt = g0 * (T(4) * eB + (eA + eC)) + g1 * (pC - pA);
                R[i] = R[i] + cx<T>{kk.x + tt.y, kk.y - tt.x};
            } else {
                R[i] = ma * (pA + pC) + mb * pB;
            }
        };
        if constexpr (RG) {
            cx<T> U[NP];
            RegionRows g = rows0;
#pragma unroll
            for (int i = 0; i < NP; ++i, g.next()) U[i] = STAGE == 1 ? x1[g.at()] : x2[g.at()];
            if constexpr (STAGE == 1) load_in(NT);
            reg_sweep<T, NP, NW, STAGE == 1>(U, edges[0], wv, rhs);
        } else {
            {
                RegionRows g = rows0;
#pragma unroll
                for (int i = 0; i < NP; ++i, g.next()) lrow(bufs[0], i) = STAGE == 1 ? x1[g.at()] : x2[g.at()];
            }
            if constexpr (STAGE == 1) load_in(NT);
            __syncthreads();
            split_sweep<T, NP, RX, STAGE == 1>(bufs[0] + r0 * RX, xm, px, xp, rhs);
        }
    }
    static_assert(MR == 0 || (STAGE == 0 && MR <= kMassRMax), "the separable mass inverse is step 1");
    if constexpr (MR > 0 && RX == kTX) {
        // a region row is one wave: the x filter by lane shifts (DPP) in registers; the y filter from the
        // thread's own rows, and from LDS for the MR rows beyond either end of its block, which the waves
        // above and below store.  Rows q in [MR, RY - MR) and columns in [MR, RX - MR) come out exact.
        static_assert(2 * MR <= NP, "a thread's block holds the rows its neighbours need");
        T w[MR + 1];
#pragma unroll
        for (int k = 0; k <= MR; ++k) w[k] = T(s.wsep[k]);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            cx<T> lo = R[i], hi = R[i];
            cx<T> acc = w[0] * R[i];
#pragma unroll
            for (int k = 1; k <= MR; ++k) {
                lo = lane_shift<kDppWaveShr1>(lo);   // column px - k
                hi = lane_shift<kDppWaveShl1>(hi);   // column px + k
                acc = acc + w[k] * (lo + hi);
            }
            X[i] = acc;
        }
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i < MR || i >= NP - MR) lrow(bufs[0], i) = X[i];
        __syncthreads();
        // (R, no longer needed, takes the y-filtered rows)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            cx<T> acc = w[0] * X[i];
#pragma unroll
            for (int k = 1; k <= MR; ++k) {
                const cx<T> a = i - k >= 0 ? X[i - k] : lrow(bufs[0], i - k);
                const cx<T> b = i + k < NP ? X[i + k] : lrow(bufs[0], i + k);
                acc = acc + w[k] * (a + b);
            }
            R[i] = acc;
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) X[i] = R[i];
    } else if constexpr (MR > 0) {
        // x filter of the thread's rows from LDS into X, written back over the region (one buffer), then the
        // y filter; region rows q in [MR, RY - MR) and columns in [MR, RX - MR) come out exact, and the
        // interior lies inside them (halo >= MR)
        T w[MR + 1];
#pragma unroll
        for (int k = 0; k <= MR; ++k) w[k] = T(s.wsep[k]);
#pragma unroll
        for (int i = 0; i < NP; ++i) lrow(bufs[0], i) = R[i];
        __syncthreads();
        const bool xin = px >= MR && px < RX - MR;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const cx<T>* row = &lrow(bufs[0], i);
            cx<T> acc = cx<T>{T(0), T(0)};
            if (xin) {
                acc = w[0] * row[0];
#pragma unroll
                for (int k = 1; k <= MR; ++k) acc = acc + w[k] * (row[-k] + row[k]);
            }
            X[i] = acc;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NP; ++i) lrow(bufs[0], i) = X[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int q = r0 + i;
            if (q < MR || q >= RY - MR) continue;
            const cx<T>* col = &lrow(bufs[0], i);
            cx<T> acc = w[0] * col[0];
#pragma unroll
            for (int k = 1; k <= MR; ++k) acc = acc + w[k] * (col[-k * RX] + col[k * RX]);
            X[i] = acc;
        }
    } else {
    // Chebyshev iterations on OP = M (stage 0) or L (stages 1, 2)
    constexpr bool isM = STAGE == 0;
    const int its = isM ? sM : sL;
    const double(*cb)[2] = sys[tile.sys].cb[isM ? 0 : 1];
    const SplitCoef oc = split_coef(s.h, isM ? 1.0 : s.isq_dt, isM ? 0.0 : s.sq_kap);
    const T oa = T(oc.a), ob = T(oc.b), occ = T(oc.c), od = T(oc.d);
    const T d0 = T(cb[0][0]);
    if constexpr (RG) {
        // d_{k-1} of the thread's rows in D; iteration k sweeps them with edge set k & 1 (set 0 also served
        // the right-hand side sweep of stages 1 and 2, whose reads finished before iteration 1's barrier) and
        // replaces each row's d once the sweep has read it
        cx<T> D[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            D[i] = d0 * R[i];
            X[i] = D[i];
        }
        auto iteration = [&](int k, auto store) {
            const T c1 = T(cb[k][0]), c2 = T(cb[k][1]);
            reg_sweep<T, NP, NW, false>(D, edges[k & 1], wv, [&](int i, cx<T> pA, cx<T> pB, cx<T> pC, cx<T> uA,
                                                                  cx<T> uB, cx<T> uC, cx<T>, cx<T>, cx<T>) {
                cx<T> q = R[i] - oa * (pA + pC) - ob * pB;
                if constexpr (!isM) q = q - occ * (uA + uC) - od * uB;
                R[i] = q;
                const cx<T> dv = c1 * uB + c2 * q;
                X[i] = X[i] + dv;
                if constexpr (decltype(store)::value) D[i] = dv;
            });
        };
        for (int k = 1; k + 1 < its; ++k) iteration(k, std::true_type{});
        if (its > 1) iteration(its - 1, std::false_type{});
    } else if constexpr (NB == 2) {
        // d_0 into bufs[1]; iteration k reads d_{k-1} from bufs[k & 1] (the barrier at its start orders it
        // after every write of d_{k-1} and after every read of the buffer it writes, bufs[(k + 1) & 1], by
        // iteration k - 1 or by the prologue of stages 1 and 2)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const cx<T> dv = d0 * R[i];
            X[i] = dv;
            lrow(bufs[1], i) = dv;
        }
        auto iteration = [&](int k, auto store) {
            __syncthreads();
            const cx<T>* b = bufs[k & 1];
            cx<T>* bn = bufs[(k + 1) & 1];
            const T c1 = T(cb[k][0]), c2 = T(cb[k][1]);
            split_sweep<T, NP, RX, false>(b + r0 * RX, xm, px, xp, [&](int i, cx<T> pA, cx<T> pB, cx<T> pC, cx<T> uA,
                                                                        cx<T> uB, cx<T> uC, cx<T>, cx<T>, cx<T>) {
                // r -= OP d_{k-1} (uB = this node's d_{k-1}), as a chain of fused multiply-adds (the mass
                // operator has no centre terms); d_k = c1 d_{k-1} + c2 r; x += d_k
                cx<T> q = R[i] - oa * (pA + pC) - ob * pB;
                if constexpr (!isM) q = q - occ * (uA + uC) - od * uB;
                R[i] = q;
                const cx<T> dv = c1 * uB + c2 * q;
                X[i] = X[i] + dv;
                if constexpr (decltype(store)::value) lrow(bn, i) = dv;
            });
        };
        // the last iteration's d is not needed by anyone: it is not stored
        for (int k = 1; k + 1 < its; ++k) iteration(k, std::true_type{});
        if (its > 1) iteration(its - 1, std::false_type{});
    } else {
        cx<T> Dd[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            Dd[i] = d0 * R[i];
            X[i] = Dd[i];
        }
        for (int k = 1; k < its; ++k) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NP; ++i) lrow(bufs[0], i) = Dd[i];
            __syncthreads();
            const T c1 = T(cb[k][0]), c2 = T(cb[k][1]);
            split_sweep<T, NP, RX, false>(bufs[0] + r0 * RX, xm, px, xp,
                                          [&](int i, cx<T> pA, cx<T> pB, cx<T> pC, cx<T> uA, cx<T> uB, cx<T> uC,
                                              cx<T>, cx<T>, cx<T>) {
                                              cx<T> q = R[i] - oa * (pA + pC) - ob * pB;
                                              if constexpr (!isM) q = q - occ * (uA + uC) - od * uB;
                                              R[i] = q;
                                              Dd[i] = c1 * Dd[i] + c2 * R[i];
                                              X[i] = X[i] + Dd[i];
                                          });
        }
    }
    }
    // output at the owned nodes
    if (!own_x) return;
    RegionRows g = rows0;
#pragma unroll
    for (int i = 0; i < NP; ++i, g.next()) {
        if (!own_row(i)) continue;
        const long long gi = g.at();
        if constexpr (STAGE == 0) {
            x1[gi] = X[i];
        } else if constexpr (STAGE == 1) {
            x2[gi] = X[i];
        } else {
            const cx<T> chi2 = X[i];
            z[gi] = x1[gi] - T(s.isq_kap) * (x2[gi] - T(s.isq_dt) * chi2);
            z[NT + gi] = chi2;
        }
    }
}

// ------------------------------------------------------------------------------------------
// The three stages in one launch, for meshes whose regions all fit on the chip at once, one per CU: a
// workgroup carries its 64 x 32 region through all of them in registers, with a halo of all their layers (9 for
// three taps and three L iterations, interior 46 x 14).  x1 and x2 never leave the workgroup and two of three
// launches go, against 3.2 times the stencil work of the interior, which counts when the regions take several rounds.
// 130 x 118 x 3 in FP32: 24.1 us in three launches, 15.8 us in one.  Steps of 24 FGMRES iterations in FP64, three
// launches and one: 252 regions (276 x 190 x 3) 1275 and 1050 us, 378 regions 1430 and 1284, 600 regions 1554 and 1653.
// ------------------------------------------------------------------------------------------
constexpr int kChebAllNP = 8, kChebAllNW = 4, kChebAllHalo = 10;

// SEP: x1 by the separable mass inverse of MR taps; else sM Chebyshev iterations (MR = 0)
template <typename T, int MR>
__global__ __launch_bounds__(64 * kChebAllNW) void k_cheb2d_all(const Sys* sys, const int* mask, const cx<T>* v, cx<T>* z,
                                                               int sM, int sL, int halo, long long NT, VIn<T> vin) {
    constexpr int NP = kChebAllNP, NW = kChebAllNW, RL = MR > 0 ? NP * NW + 2 * MR : 1;
    __shared__ cx<T> edges[2][NW][2][kTX];
    __shared__ cx<T> rows[RL * kTX];   // region rows with MR rows of padding above and below (mass filter)
    const int si = blockIdx.y, wv = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    if (mask && !mask[si]) return;
    const Sys& s = sys[si];
    Region<NP, NW> reg;
    if (!reg.init(s, halo)) return;
    int e = 0;
    cx<T> R[NP], B2[NP], X1[NP], X2[NP], D[NP];
    auto load_in = [&](long long hoff, cx<T> (&out)[NP]) {
        RegionRows g = reg.rows0;
        if (!vin.src) {
#pragma unroll
            for (int i = 0; i < NP; ++i, g.next()) out[i] = v[hoff + g.at()];
            return;
        }
        const double* hc = vin.hcoef + (long long)si * vin.hld;
        const double sc = vin.scale[si];
        zd u[NP];
        long long gi[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i, g.next()) {
            gi[i] = hoff + g.at();
            u[i] = ld<double>(vin.src, gi[i]);
        }
        for (int l = 0; l < vin.nv; ++l) {
            const zd c{hc[2 * l], hc[2 * l + 1]};
            const cx<T>* Vl = vin.V + l * vin.vs;
#pragma unroll
            for (int i = 0; i < NP; ++i) u[i] = u[i] - cmul(c, ld<double>(Vl, gi[i]));
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            out[i] = cx<T>{T(sc * u[i].x), T(sc * u[i].y)};
            if (reg.owned(i)) vin.vout[gi[i]] = out[i];
        }
    };
    // its Chebyshev iterations on OP = M or L from zero for the right-hand side R, into X
    auto cheb = [&](auto mc, int its, cx<T> (&X)[NP]) {
        constexpr bool isM = decltype(mc)::value;
        const double(*cb)[2] = s.cb[isM ? 0 : 1];
        const SplitCoef oc = split_coef(s.h, isM ? 1.0 : s.isq_dt, isM ? 0.0 : s.sq_kap);
        const T oa = T(oc.a), ob = T(oc.b), occ = T(oc.c), od = T(oc.d), d0 = T(cb[0][0]);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            D[i] = d0 * R[i];
            X[i] = D[i];
        }
        for (int k = 1; k < its; ++k) {
            const T c1 = T(cb[k][0]), c2 = T(cb[k][1]);
            reg_sweep<T, NP, NW, false>(D, edges[e], wv, [&](int i, cx<T> pA, cx<T> pB, cx<T> pC, cx<T> uA, cx<T> uB,
                                                             cx<T> uC, cx<T>, cx<T>, cx<T>) {
                cx<T> q = R[i] - oa * (pA + pC) - ob * pB;
                if constexpr (!isM) q = q - occ * (uA + uC) - od * uB;
                R[i] = q;
                const cx<T> dv = c1 * uB + c2 * q;
                X[i] = X[i] + dv;
                D[i] = dv;
            });
            e ^= 1;
        }
    };
    load_in(0, R);
    load_in(NT, B2);
    // step 1
    if constexpr (MR > 0) {
        static_assert(2 * MR <= NP, "a thread's block holds the rows its neighbours need");
        auto row = [&](int i) -> cx<T>& { return rows[(wv * NP + MR + i) * kTX + lane]; };
        // the padding only feeds the outermost halo rows
        for (int q = threadIdx.x; q < MR * kTX; q += 64 * NW) rows[q] = rows[(RL - MR) * kTX + q] = cx<T>{T(0), T(0)};
        T w[MR + 1];
#pragma unroll
        for (int k = 0; k <= MR; ++k) w[k] = T(s.wsep[k]);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            cx<T> lo = R[i], hi = R[i], acc = w[0] * R[i];
#pragma unroll
            for (int k = 1; k <= MR; ++k) {
                lo = lane_shift<kDppWaveShr1>(lo);
                hi = lane_shift<kDppWaveShl1>(hi);
                acc = acc + w[k] * (lo + hi);
            }
            D[i] = acc;
            if (i < MR || i >= NP - MR) row(i) = acc;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            cx<T> acc = w[0] * D[i];
#pragma unroll
            for (int k = 1; k <= MR; ++k) {
                const cx<T> a = i - k >= 0 ? D[i - k] : row(i - k);
                const cx<T> b = i + k < NP ? D[i + k] : row(i + k);
                acc = acc + w[k] * (a + b);
            }
            X1[i] = acc;
        }
    } else {
        cheb(std::true_type{}, sM, X1);
    }
    // step 2
    {
        const T k3 = T(s.kappa / 3.0), k4 = T(4.0 * s.kappa), kap = T(s.kappa);
        const T g0 = T(s.kappa * s.h / 6.0 * s.kv[0]), g1 = T(s.kappa * s.h / 6.0 * s.kv[1]);
        reg_sweep<T, NP, NW, true>(X1, edges[e], wv, [&](int i, cx<T> pA, cx<T> pB, cx<T> pC, cx<T> uA, cx<T> uB, cx<T> uC,
                                                         cx<T> eA, cx<T> eB, cx<T> eC) {
            const cx<T> kk = kap * (uA + uC) + k4 * uB - k3 * ((pA + pC) + pB);
            const cx<T> tt = g0 * (T(4) * eB + (eA + eC)) + g1 * (pC - pA);
            R[i] = B2[i] + cx<T>{kk.x + tt.y, kk.y - tt.x};
        });
        e ^= 1;
    }
    cheb(std::false_type{}, sL, X2);
    // steps 3 and 4
    {
        const SplitCoef m = split_coef(s.h, 1.0, 0.0);
        const T ma = T(m.a), mb = T(m.b);
        reg_sweep<T, NP, NW, false>(X2, edges[e], wv, [&](int i, cx<T> pA, cx<T> pB, cx<T> pC, cx<T>, cx<T>, cx<T>, cx<T>,
                                                          cx<T>, cx<T>) { R[i] = ma * (pA + pC) + mb * pB; });
        e ^= 1;
    }
    cx<T>(&chi2)[NP] = B2;
    cheb(std::false_type{}, sL, chi2);
    RegionRows g = reg.rows0;
#pragma unroll
    for (int i = 0; i < NP; ++i, g.next())
        if (reg.owned(i)) {
            const long long gi = g.at();
            z[gi] = X1[i] - T(s.isq_kap) * (X2[i] - T(s.isq_dt) * chi2[i]);
            z[NT + gi] = chi2[i];
        }
}

// Halo and grid of k_cheb2d_all; grid.x = 0 where it does not apply.
static dim3 cheb_all_grid(const Dev& d, int mass_iters, int diff_iters, int mass_sep, int& halo) {
    halo = (mass_sep > 0 ? mass_sep : mass_iters - 1) + 2 * diff_iters;
    if (halo > kChebAllHalo) return dim3(0);
    const int IX = kTX - 2 * halo, IY = kChebAllNP * kChebAllNW - 2 * halo;
    const long long n = (long long)((d.maxn[0] + IX - 1) / IX) * ((d.maxn[1] + IY - 1) / IY);
    return n * d.S <= d.cus ? dim3((unsigned)n, d.S) : dim3(0);
}

template <typename T, int RX, int RY, int NTH>
static void cheb_stages(const Dev& d, const CTile* ctiles, int nctiles, int halo, const cx<T>* v, cx<T>* z,
                        cx<T>* x1, cx<T>* x2, int mass_iters, int diff_iters, int mass_sep, const VIn<T>& vin,
                        const int* mask, hipStream_t st) {
    const dim3 g(nctiles), b(NTH);
    // input half read (v, or the vectors the basis vector is formed from) and then the basis vector written
    const double pts = (double)d.NT, in = (double)sizeof(cx<T>) * (vin.src ? 1 + vin.nv : 1),
                 vb = vin.src ? (double)sizeof(cx<T>) : 0.0;
    {
        ProbeScope ps(d, KID_CHEB, st, pts * (in + sizeof(cx<T>) + vb), mask, true);
        auto stage0 = [&](auto mr) {
            ps.launch(k_cheb2d<T, 0, RX, RY, NTH, decltype(mr)::value>, g, b, d.sys, ctiles, mask, v, x1, x2, z,
                      mass_iters, diff_iters, halo, d.NT, vin);
        };
        static_assert(kMassRMax == 4, "one case per tap count");
        switch (mass_sep) {
            case 0: stage0(std::integral_constant<int, 0>{}); break;
            case 1: stage0(std::integral_constant<int, 1>{}); break;
            case 2: stage0(std::integral_constant<int, 2>{}); break;
            case 3: stage0(std::integral_constant<int, 3>{}); break;
            default: stage0(std::integral_constant<int, 4>{}); break;
        }
    }
    {
        ProbeScope ps(d, KID_CHEB, st, pts * (in + 2 * sizeof(cx<T>) + vb), mask, true);
        ps.launch(k_cheb2d<T, 1, RX, RY, NTH>, g, b, d.sys, ctiles, mask, v, x1, x2, z, mass_iters, diff_iters, halo,
                  d.NT, vin);
    }
    ProbeScope ps(d, KID_CHEB, st, pts * 4 * sizeof(cx<T>), mask, true);
    ps.launch(k_cheb2d<T, 2, RX, RY, NTH>, g, b, d.sys, ctiles, mask, v, x1, x2, z, mass_iters, diff_iters, halo,
              d.NT, VIn<T>{});
}

template <typename T>
void launch_precond_cheb(const Dev& d, int shape, const CTile* ctiles, int nctiles, int halo, const cx<T>* v,
                         cx<T>* z, cx<T>* x1, cx<T>* x2, int mass_iters, int diff_iters, int mass_sep,
                         const VIn<T>& vin, const int* mask, hipStream_t st) {
    int halo_all = 0;
    // with many basis vectors the halo's share of their loads outweighs the saved launches
    const dim3 all = vin.nv <= 8 && !d.cheb_stages ? cheb_all_grid(d, mass_iters, diff_iters, mass_sep, halo_all) : dim3(0);
    if (all.x > 0) {
        const double c = sizeof(cx<T>), in = c * (vin.src ? 2 + vin.nv : 1);
        ProbeScope ps(d, KID_CHEB, st, (double)d.NT * 2.0 * (in + c), mask, true);
        auto go = [&](auto mr) {
            ps.launch(k_cheb2d_all<T, decltype(mr)::value>, all, dim3(64 * kChebAllNW), d.sys, mask, v, z, mass_iters,
                      diff_iters, halo_all, d.NT, vin);
        };
        static_assert(kMassRMax == 4, "one case per tap count");
        switch (mass_sep) {
            case 0: go(std::integral_constant<int, 0>{}); break;
            case 1: go(std::integral_constant<int, 1>{}); break;
            case 2: go(std::integral_constant<int, 2>{}); break;
            case 3: go(std::integral_constant<int, 3>{}); break;
            default: go(std::integral_constant<int, 4>{}); break;
        }
        return;
    }
#define APFC_CHEB_SHAPE(I)                                                                                       \
    case I:                                                                                                      \
        cheb_stages<T, kChebShape[I][0], kChebShape[I][1], kChebShape[I][2]>(                                    \
            d, ctiles, nctiles, halo, v, z, x1, x2, mass_iters, diff_iters, mass_sep, vin, mask, st);               \
        break;
    static_assert(kChebShapes == 6, "one case per region shape");
    switch (shape) {
        APFC_CHEB_SHAPE(1)
        APFC_CHEB_SHAPE(2)
        APFC_CHEB_SHAPE(3)
        APFC_CHEB_SHAPE(4)
        APFC_CHEB_SHAPE(5)
        default: cheb_stages<T, kChebShape[0][0], kChebShape[0][1], kChebShape[0][2]>(
            d, ctiles, nctiles, halo, v, z, x1, x2, mass_iters, diff_iters, mass_sep, vin, mask, st);
    }
#undef APFC_CHEB_SHAPE
}
template void launch_precond_cheb<double>(const Dev&, int, const CTile*, int, int, const zd*, zd*, zd*, zd*, int, int,
                                          int, const VIn<double>&, const int*, hipStream_t);
template void launch_precond_cheb<float>(const Dev&, int, const CTile*, int, int, const zf*, zf*, zf*, zf*, int, int,
                                         int, const VIn<float>&, const int*, hipStream_t);

}  // namespace apfc
