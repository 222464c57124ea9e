// Linear-model rollout + cost with full weights Q, R, Qf (eq. 3 in general
// form) on the matrix cores (gfx950).
//
// A tile of 16 candidates runs on NT = ceil(n / 16) wavefronts, wavefront w
// owning state rows 16w .. 16w+15, in the layout, K order and exchange of the
// M-split rollout (rollout_linear.hpp).  The weight product Q x_k is a second
// contraction over the same B operands as A_d x_k: its 4 NT MFMAs per step
// depend on nothing in the step, so they run while the new state's sums
// finish and go through LDS.  The stage cost is (x - g)^T Q (x - g): with one
// M-tile the product takes x - g itself, with more it is Q x - Q g, Q g
// precomputed; at x_T, Q (x - g) always.  The diagonal of A_d is left out of the
// operands and added last, by one fused operation: near the identity the terms
// after it would round by the state's own size (FP32, error of the cost
// relative to the vector-ALU form, spring chains of 2 to 30 DoF: 0.65 to 1.18
// with the diagonal in its K slice, 0.26 to 0.68 this way, for 2 to 7 % of the
// time; states around a goal 100 units away 0.51 to 1.12, now 0.30 to 0.84).  The
// input cost of a knot segment is closed form in
// E_a = U_a - u_g and R E_a, one product per knot:
//   S00 E_a^T R E_a + 2 S01 E_a^T R E_b + S11 E_b^T R E_b
// with the sums of (1-c)^2, c (1-c), c^2 over the segment.  The terminal
// weight's operands are loaded after the last step.
//
// The step's chain of MFMAs bounds it (8 NT of them, 32 cycles each in FP32).
// On the vector ALUs, 16 lanes per candidate with A_d and Q read from LDS in
// every step, the 7-DoF chain (4096 candidates, 50 steps, FP32) took 40 us;
// here 17.4 us; 32 DoF 245 and 54 us; FP64 47 and 29, 322 and 93 us.
#pragma once
#include <math.h>

#include "internal.hpp"
#include "mfma.hpp"

namespace empc {

// LV: live K slices of a single M-tile (states 4 v .. 4 v + 3 of slice v; 4
// with more M-tiles): FP64 n = 4, 256 candidates, 50 steps 25.4 us with all
// four slices, 15.5 us with one.
template <typename T, int NT, int NU, bool BOX, int LV = 4>
__global__ __launch_bounds__(64 * NT) void roll_linear_full(ProbView<T> P,
                                                            const T *__restrict__ x0,
                                                            const T *__restrict__ knots,
                                                            int64_t ld, int64_t ncand,
                                                            T *__restrict__ cost) {
    typedef typename Mfma<T>::v4 v4;
    constexpr int UT = (NU + 3) / 4, UW = (UT + NT - 1) / NT;  // input tiles: in all, per wavefront
    __shared__ v4 xs[2][NT][64];
    __shared__ T part[NT][16];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int64_t cand = xcd_swizzle(blockIdx.x, gridDim.x) * 16 + col;
    const bool valid = cand < ncand;
    const int64_t cand_c = valid ? cand : ncand - 1;
    const int n = P.n, m = P.m, p = P.p, Tn = P.Tn;
    const int arow = 16 * w + Mfma<T>::mstate(col);

    // knots a, b = a + 1 and a + 2 while segment a runs: lane (grp, col) of
    // slice s holds input 4 s + grp (padded inputs meet zero operands)
    T Ka[NU], Kb[NU], Kn[NU];
    auto load_knot = [&](int j, T *U) {
        const int kc = j < p ? j : p - 1;
#pragma unroll
        for (int s = 0; s < NU; ++s) {
            const int i = 4 * s + grp;
            U[s] = knots[(int64_t)(kc * m + (i < m ? i : m - 1)) * ld + cand_c];
        }
    };
    load_knot(0, Ka);
    load_knot(1, Kb);
    // operands by slot i (M-tile t = (w + i) mod NT); full or diagonal weights
    auto q_at = [&](int row, int kk) { return P.Qm ? P.Qm[row * n + kk] : row == kk ? P.q[row] : (T)0; };
    T aX[4 * NT], aQ[4 * NT], aU[NU], aR[UW][NU], Ug[NU];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int kk = 16 * ((w + i) % NT) + Mfma<T>::row(grp, v);
            const bool in = arow < n && kk < n;
            aX[4 * i + v] = in && arow != kk ? P.Ad[arow * n + kk] : (T)0;  // diagonal apart
            aQ[4 * i + v] = in ? q_at(arow, kk) : (T)0;
        }
#pragma unroll
    for (int s = 0; s < NU; ++s) {
        const int j = 4 * s + grp;
        aU[s] = arow < n && j < m ? P.Bd[arow * m + j] : (T)0;
        Ug[s] = j < m && P.ug ? P.ug[j] : (T)0;
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            const int row = 16 * (w + NT * u) + Mfma<T>::mstate(col);
            aR[u][s] = row >= m || j >= m ? (T)0
                       : P.Rm             ? P.Rm[row * m + j]
                       : row == j         ? P.r[row]
                                          : (T)0;
        }
    }
    v4 X, Wd, Xg, Diag, Lo, Hi, Pn = {0, 0, 0, 0}, Cn = {0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = 16 * w + Mfma<T>::row(grp, v);
        const bool in = row < n;
        X[v] = in ? x0[row] : (T)0;
        Wd[v] = in && P.wd ? P.wd[row] : (T)0;
        Xg[v] = in && P.xg ? P.xg[row] : (T)0;
        Diag[v] = in ? P.Ad[row * n + row] : (T)0;
        Lo[v] = BOX && in ? P.xlo[row] : (T)-1;  // padding rows: around their zero state
        Hi[v] = BOX && in ? P.xhi[row] : (T)1;
    }
    // all of the model is waited for here, before the step loop's prefetches
    __builtin_amdgcn_s_waitcnt(VMCNT0);
    // this wavefront's rows of M V over all M-tiles (own tile first), from
    // `start`, even and odd slices in two chains
    auto contract = [&](const T *op, const v4 *V, v4 start) {
        v4 acc[2] = {start, v4{0, 0, 0, 0}};
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < LV; ++v)
                acc[v & 1] = Mfma<T>::op(op[4 * i + v], V[i][v], acc[v & 1]);
        return LV == 1 ? acc[0] : acc[0] + acc[1];
    };
    // stored own tile -> every tile, by slot
    auto gather = [&](int b, v4 *V) {
        V[0] = X;
        if (NT == 1) return;
        lds_barrier();
#pragma unroll
        for (int i = 1; i < NT; ++i) V[i] = xs[b][(w + i) % NT][lane];
    };
    auto response = [&](const T *U) {
        v4 V[2] = {Wd, v4{0, 0, 0, 0}};
#pragma unroll
        for (int s = 0; s < NU; ++s) V[s & 1] = Mfma<T>::op(aU[s], U[s], V[s & 1]);
        return V[0] + V[1];
    };
    // R (U - u_g), rows of this wavefront's input tiles
    auto r_times = [&](const T *U, v4 *RE) {
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            v4 V[2] = {v4{0, 0, 0, 0}, v4{0, 0, 0, 0}};
#pragma unroll
            for (int s = 0; s < NU; ++s) V[s & 1] = Mfma<T>::op(aR[u][s], U[s] - Ug[s], V[s & 1]);
            RE[u] = V[0] + V[1];
        }
    };
    // the inputs of this wavefront's tile u, register v (slice 4 (w + NT u) + v)
    auto input_of = [&](const T *U, int u, int v) -> T {
        T e = 0;
#pragma unroll
        for (int t = 0; t < UT; ++t)
            if (4 * t + v < NU && t == w + NT * u) e = U[4 * t + v] - Ug[4 * t + v];
        return e;
    };
    // Q g, from the goal published like a state
    v4 V[NT], Qg;
    if constexpr (NT > 1) {
        const v4 x = X;
        X = Xg;
        xs[1][w][lane] = X;
        gather(1, V);
        Qg = contract(aQ, V, v4{0, 0, 0, 0});
        X = x;
        xs[0][w][lane] = X;
    }
    v4 Va = response(Ka), Vb = response(Kb), REa[UW], REb[UW];
    r_times(Ka, REa);
    r_times(Kb, REb);
    const T inv_den = Tn > 1 ? (T)1 / (T)(Tn - 1) : (T)0;
    // Stage costs summed per state row: one running sum over a lane's four rows
    // rounds four times as often (FP32, n = 14, 400 steps: rms relative error
    // 2.2e-7 that way, 1.0e-7 per row), for 2 to 4 % of the time
    v4 Js = {0, 0, 0, 0};
    T J = 0;
    int buf = 0, k = 0;
    for (int a = 0; a < p; ++a) {
        // first step of segment a + 1
        const int kend =
            p == 1 || a == p - 1 ? Tn : ((a + 1) * (Tn - 1) + (p - 2)) / (p - 1);
        load_knot(a + 2, Kn);
        const v4 dV = Vb - Va;
        T s00 = 0, s01 = 0, s11 = 0;
        int rem = k * (p - 1) - a * (Tn - 1);
        for (; k < kend; ++k, rem += p - 1) {
            const T c = (T)rem * inv_den, d = (T)1 - c;
            s00 += d * d;
            s01 += c * d;
            s11 += c * c;
            gather(buf, V);
            const v4 Xk = X;
            X = contract(aX, V, v4{0, 0, 0, 0}) + (Va + c * dV);
#pragma unroll
            for (int v = 0; v < LV; ++v) X[v] += Diag[v] * Xk[v];
            buf ^= 1;
            if (NT > 1) xs[buf][w][lane] = X;
            // stage cost of x_k (x_0 has none), beside the new state's way
            const v4 E = Xk - Xg;
            v4 QE;
            if constexpr (NT == 1)
                QE = contract(aQ, &E, v4{0, 0, 0, 0});
            else
                QE = contract(aQ, V, -Qg);
#pragma unroll
            for (int v = 0; v < LV; ++v)
                Js[v] = k > 0 ? Js[v] + E[v] * QE[v] : (T)0;
            if (BOX) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {  // x_{k+1}'s
                    Pn[v] += box_pen(X[v], Lo[v], Hi[v]);
                    Cn[v] += box_out(X[v], Lo[v], Hi[v]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UW; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const T ea = input_of(Ka, u, v), eb = a == p - 1 ? (T)0 : input_of(Kb, u, v);
                const T rb = a == p - 1 ? (T)0 : REb[u][v];
                J += s00 * ea * REa[u][v] + (T)2 * s01 * ea * rb + s11 * eb * rb;
            }
        Va = Vb;
#pragma unroll
        for (int u = 0; u < UW; ++u) REa[u] = REb[u];
#pragma unroll
        for (int s = 0; s < NU; ++s) {
            Ka[s] = Kb[s];
            Kb[s] = Kn[s];
        }
        if (a + 1 < p) {
            Vb = response(Kb);
            r_times(Kb, REb);
        }
    }
    // x_T: stage and terminal weight of E = x_T - g, published like a state (not
    // Q x - Q g: at a state near a goal far from the origin, where x_T is meant
    // to be, the two cancel)
    const v4 E = X - Xg;
    {
        const v4 x = X;
        X = E;
        // over this wavefront's tile of x_T, which no other has read (the other
        // buffer is the one that they may still be reading)
        if (NT > 1) xs[buf][w][lane] = X;
        gather(buf, V);
        X = x;
    }
    const v4 QE = contract(aQ, V, v4{0, 0, 0, 0});
    v4 F = {0, 0, 0, 0};
    if (P.Qfm) {
        T aF[4 * NT];
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int kk = 16 * ((w + i) % NT) + Mfma<T>::row(grp, v);
                aF[4 * i + v] = arow < n && kk < n ? P.Qfm[arow * n + kk] : (T)0;
            }
        F = contract(aF, V, v4{0, 0, 0, 0});
    } else if (P.qf) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * w + Mfma<T>::row(grp, v);
            F[v] = row < n ? P.qf[row] * E[v] : (T)0;
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        J += Js[v] + E[v] * (QE[v] + F[v]);
        if (BOX) {
            const int row = 16 * w + Mfma<T>::row(grp, v);
            const bool in = row < n;
            J += (in ? P.qb[row] : (T)0) * Pn[v] + (in && P.sb ? P.sb[row] : (T)0) * Cn[v];
        }
    }
    J += __shfl_xor(J, 16, 64);
    J += __shfl_xor(J, 32, 64);
    if (NT > 1) {
        if (grp == 0) part[w][col] = J;
        lds_barrier();
        J = part[0][col];
#pragma unroll
        for (int i = 1; i < NT; ++i) J += part[i][col];
    }
    if (w == 0 && grp == 0 && valid) cost[cand] = J;
}

}  // namespace empc
