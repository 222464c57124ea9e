// Adjoint gradient and Adam refinement of the linear model on the matrix
// cores (gfx950), shared by the FP32 and FP64 translation units.
//
// A tile of 16 candidates runs on a workgroup of NT = ceil(n / 16) state
// wavefronts, wavefront w owning state rows 16w .. 16w+15, in the accumulator
// layout and K order of the M-split rollout (rollout_linear.hpp), and of UT =
// ceil(m / 16) input wavefronts.  The backward recursion lambda_k =
// 2 Q (x_k - g) + A^T lambda_{k+1} is the same contraction with A transposed,
// so the adjoint chains through the accumulators as the state does.  The input
// wavefronts do what hangs on the inputs beside that chain: forward the products
// B_d u_k + w_d, one step ahead, and the input cost; backward the products
// B_d^T lambda_{k+1} and their sums over the knots.  The tile's knots sit in
// LDS, and so do the states of the forward pass: all of them when they fit (2 T
// dependent steps), else one per block of S steps, each block recomputed before
// it is walked backward (3 T steps).
//
// What bounds it is the chain of dependent steps (4 NT MFMAs in four chains, an
// LDS round trip and a barrier each), as in the M-split rollout: one
// wavefront pair per candidate took the same chain for a single candidate.
// 14-DoF chain, T = 50, p = 10, FP32, 4096 candidates: 236 us with a workgroup
// per candidate on the vector ALUs, 45 us here (65536, in blocks: 3.1 ms and 0.47
// ms); 64 candidates with five Adam steps: 236 and 228 us.
// Products with B_d per knot instead of per step, blended (41 us, 202 us), lost
// accuracy: see drive.  Errors against 64 bits, relative to the per-candidate
// kernel's (FP32, rms over horizons of 20 to 200): gradient 0.89 to 1.00 and cost
// 0.92 to 0.98 for random models of 14 to 60 states, 0.52 to 0.69 and 0.60 to 0.79
// for spring chains of 2 to 30 DoF (see the diagonal below).
#pragma once
#include <math.h>

#include <algorithm>

#include "internal.hpp"
#include "mfma.hpp"

namespace empc {

// LDS plan (element counts) and the way the states are kept.
struct LinAdjPlan {
    int full;          // every state kept
    int S, nblk;       // steps per block and blocks (full: one block)
    size_t oX, oL, oD, oR, oQ, oC, oU, oM1, oM2, oG, total;
};
inline LinAdjPlan lin_adj_layout(int NT, int UT, int T, int p, bool refine, int S, bool full) {
    LinAdjPlan g;
    g.full = full;
    g.S = S;
    g.nblk = full ? 1 : (T + S - 1) / S;
    const size_t slot = (size_t)NT * 256, kn = (size_t)p * UT * 256;
    size_t o = 0;
    // full: x_0 .. x_{T-1}; else the blocks' first states and one block
    g.oX = o; o += slot * (full ? (size_t)T : (size_t)g.nblk + S);
    g.oL = o; o += 2 * slot;
    g.oD = o; o += 2 * slot;
    g.oU = o; o += kn;
    g.oM1 = o; o += refine ? kn : 0;
    g.oM2 = o; o += refine ? kn : 0;
    g.oG = o; o += refine ? kn : 0;
    g.oR = o; o += (size_t)(NT + UT) * 16;
    g.oQ = o; o += (size_t)NT * 16;
    g.oC = o; o += (size_t)T + 1;
    g.total = o;
    return g;
}

template <typename T, int NT, int UT>
__global__ __launch_bounds__(64 * (NT + UT)) void adjoint_linear_kernel(
    ProbView<T> P, LinAdjPlan G, const T *__restrict__ x0, const T *__restrict__ knots,
    int64_t ncand, int64_t ld, T *__restrict__ dJ, T *__restrict__ cost, int steps, T lr,
    T *__restrict__ knots_io, T *__restrict__ cost_io) {
    typedef typename Mfma<T>::v4 v4;
    constexpr int NU = 4 * UT, KN = NU * 64;  // input slices; elements of one knot
    constexpr int NW = NT + UT;  // state wavefronts, input wavefronts
    extern __shared__ __align__(32) unsigned char adj_smem[];
    T *sm = (T *)adj_smem;
    T *sU = sm + G.oU, *sC = sm + G.oC, *sR = sm + G.oR;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int64_t cand = xcd_swizzle(blockIdx.x, gridDim.x) * 16 + col;
    const bool valid = cand < ncand, refine = steps > 0;
    const int n = P.n, m = P.m, p = P.p, Tn = P.Tn;
    const bool box = P.qb != nullptr;  // uniform
    const int arow = Mfma<T>::mstate(col);

    // the tile's knots, [knot][slice][lane]: lane (grp, col) of slice s holds
    // input 4 s + grp of candidate col (past m or the candidates: a value
    // that is never stored and meets zero weights)
    const T *src = refine ? knots_io : knots;
    const int64_t cand_c = valid ? cand : ncand - 1;
    constexpr int LB = 16;
    for (int e0 = w; e0 < p * NU; e0 += LB * NW) {
        T b[LB];
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            const int e = min(e0 + q * NW, p * NU - 1), i = 4 * (e % NU) + grp;
            b[q] = src[(int64_t)((e / NU) * m + min(i, m - 1)) * ld + cand_c];
        }
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            const int e = e0 + q * NW;
            if (e < p * NU) sU[e * 64 + lane] = 4 * (e % NU) + grp < m ? b[q] : (T)0;
        }
    }
    if (refine)
        for (int e = threadIdx.x; e < p * KN; e += 64 * NW) sm[G.oM1 + e] = sm[G.oM2 + e] = 0;
    // first step of segment a (steps with idx1 = a)
    auto seg_start = [&](int a) {
        return p == 1 ? (a == 0 ? 0 : Tn) : a >= p ? Tn : (a * (Tn - 1) + p - 2) / (p - 1);
    };
    // the steps' blend weights c_k (divided: a rounded reciprocal would scale all
    // of them alike)
    for (int k = threadIdx.x; k <= Tn; k += 64 * NW) {
        const Knot kn = knot_at(Tn, p, min(k, Tn - 1));
        sC[k] = (T)kn.rem / (T)kn.den;
    }
    auto tile = [&](T *slot, int t) { return reinterpret_cast<v4 *>(slot) + t * 64 + lane; };
    auto slot = [&](int k) { return sm + G.oX + (size_t)k * NT * 256; };
    auto lam_at = [&](int i) { return sm + G.oL + i * (NT * 256); };    // rings of two
    auto drive_at = [&](int i) { return sm + G.oD + i * (NT * 256); };
    const v4 zero = {0, 0, 0, 0};

    // Operands of input wavefront q: it multiplies by the rows of B_d of M-tiles
    // q, q + UT, .. and by the rows q of B_d^T
    constexpr int NB = (NT + UT - 1) / UT;
    struct Inputs {
        int q;
        T bT[4 * NT];     // rows of B_d^T of output tile q, by M-tile
        T b[NB][NU];      // rows of B_d of M-tile q + UT i, by input slice
        v4 Wd[NB];
        T Rw[4], Ug[4];   // register s: input 16 q + 4 s + grp
    };
    auto load_inputs = [&](Inputs &I) __attribute__((always_inline)) {
        I.q = w - NT;
#pragma unroll
        for (int e = 0; e < 4 * NT; ++e) {
            const int row = 16 * I.q + arow, kk = 16 * (e / 4) + Mfma<T>::row(grp, e % 4);
            I.bT[e] = row < m && kk < n ? P.Bd[kk * m + row] : (T)0;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int t = I.q + UT * i;
#pragma unroll
            for (int s = 0; s < NU; ++s) {
                const int row = 16 * t + arow, j = 4 * s + grp;
                I.b[i][s] = row < n && j < m ? P.Bd[row * m + j] : (T)0;
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * t + Mfma<T>::row(grp, v);
                I.Wd[i][v] = row < n && P.wd ? P.wd[row] : (T)0;
            }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int i = 16 * I.q + 4 * s + grp;
            I.Rw[s] = i < m ? P.r[i] : (T)0;
            I.Ug[s] = i < m && P.ug ? P.ug[i] : (T)0;
        }
    };
    // the knot's inputs, from slice s0 on
    auto knot = [&](int j, int s0, auto &U) __attribute__((always_inline)) {
        const T *u = sU + (size_t)(j < p ? j : p - 1) * KN + 64 * s0 + lane;
#pragma unroll
        for (int s = 0; s < (int)(sizeof(U) / sizeof(T)); ++s) U[s] = u[64 * s];
    };
    // B_d u_k + w_d, rows of the wavefront's i-th M-tile.  A product per step: from
    // products per knot, blended, the steps of a segment would share two vectors'
    // rounding, a constant force (states 100 times as far from the origin as from
    // the goal, 28 states, FP32: gradient error 4.5e-6 against 6e-7).
    auto drive = [&](const Inputs &I, const T *u, int i) __attribute__((always_inline)) {
        v4 acc[4] = {I.Wd[i], zero, zero, zero};
#pragma unroll
        for (int s = 0; s < NU; ++s) acc[s & 3] = Mfma<T>::op(I.b[i][s], u[s], acc[s & 3]);
        return (acc[0] + acc[1]) + (acc[2] + acc[3]);
    };
    // dJ/dU_j: to dJ, or to G when refining.  The sums over the steps that lead to
    // it, and those of the cost, are in FP64: their rounding is the result's own.
    typedef Mfma<double>::v4 d4;
    auto knot_done = [&](const Inputs &I, int j, const d4 &sum) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int i = 16 * I.q + 4 * s + grp;
            if (refine)
                sm[G.oG + (size_t)j * KN + 256 * I.q + 64 * s + lane] = (T)sum[s];
            else if (i < m && valid)
                dJ[(int64_t)(j * m + i) * ld + cand] = (T)sum[s];
        }
    };
    // the wavefronts' shares of the cost, summed in FP64: what is added at the
    // cost's own size is rounded once
    auto total = [&]() __attribute__((always_inline)) -> T {
        double J = sR[col];
#pragma unroll
        for (int t = 1; t < NT + UT; ++t) J += sR[t * 16 + col];
        return (T)J;
    };
    auto over_rows = [&](double J) __attribute__((always_inline)) {  // the four lanes of a candidate
        J += __shfl_xor(J, 16, 64);
        return J + __shfl_xor(J, 32, 64);
    };

    // The passes of one side: forward() (the cost, in every lane) and backward()
    // (the gradient, to dJ or to G).  Both sides pass the same barriers: one per
    // step of a march, one in forward() after it, one per backward step.
    auto passes = [&](auto &&forward, auto &&backward, bool writes_cost)
                      __attribute__((always_inline)) {
        lds_barrier();  // knots, sums
        if (!refine) {
            const T J = forward();
            if (cost && writes_cost && grp == 0 && valid) cost[cand] = J;
            backward();
            return;
        }
        // Adam (Kingma & Ba 2015), bias-corrected, clamp after each update
        const T b1 = (T)0.9, b2 = (T)0.999, eps = (T)1e-8;
        T b1t = 1, b2t = 1, J0 = 0;
        for (int t = 1; t <= steps; ++t) {
            const T Jt = forward();
            if (t == 1) J0 = Jt;
            backward();
            lds_barrier();
            b1t *= b1;
            b2t *= b2;
            for (int e = threadIdx.x; e < p * KN; e += 64 * NW) {
                const int i = 4 * (e / 64 % NU) + grp;
                if (i >= m) continue;
                const T g = sm[G.oG + e];
                const T m1 = b1 * sm[G.oM1 + e] + ((T)1 - b1) * g;
                const T m2 = b2 * sm[G.oM2 + e] + ((T)1 - b2) * g * g;
                sm[G.oM1 + e] = m1;
                sm[G.oM2 + e] = m2;
                const T mh = m1 / ((T)1 - b1t), vh = m2 / ((T)1 - b2t);
                T U = sU[e] - lr * mh / (sqrt(vh) + eps);
                U = U < P.umin[i] ? P.umin[i] : U;
                U = U > P.umax[i] ? P.umax[i] : U;
                sU[e] = U;
            }
            lds_barrier();
        }
        // accept the refined knots only if they cost less, both costs by this pass
        const T Jn = forward();
        if (valid && Jn < J0) {
            for (int e = w; e < p * NU; e += NW) {
                const int i = 4 * (e % NU) + grp;
                if (i < m) knots_io[(int64_t)((e / NU) * m + i) * ld + cand] = sU[e * 64 + lane];
            }
            if (writes_cost && grp == 0) cost_io[cand] = Jn;
        }
    };

    if (w >= NT) {
        // An input wavefront.  Forward, it stays one step ahead and leaves the
        // steps' B_d u_k + w_d in a ring of two; backward, it multiplies the
        // lambda that the state wavefronts exchange and weights the product into
        // the sums of the step's two knots.
        Inputs I;
        load_inputs(I);
        auto march = [&](int k0, int k1, auto &&each) __attribute__((always_inline)) {
            if (k0 >= k1) return;
            int a = p == 1 || Tn == 1 ? 0 : k0 * (p - 1) / (Tn - 1), ke = seg_start(a + 1);
            T Ua[NU], Ub[NU];  // knots a and a + 1
            knot(a, 0, Ua);
            knot(a + 1, 0, Ub);
            T c = sC[k0];
            for (int k = k0; k < k1; ++k) {
                T u[NU];
#pragma unroll
                for (int s = 0; s < NU; ++s) u[s] = ((T)1 - c) * Ua[s] + c * Ub[s];
                c = sC[k + 1];
                each(u, k + 1 == ke);
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    if (I.q + UT * i < NT)  // uniform
                        *tile(drive_at(k & 1), I.q + UT * i) = drive(I, u, i);
                lds_barrier();
                if (k + 1 == ke) {
                    ++a;
                    ke = seg_start(a + 1);
#pragma unroll
                    for (int s = 0; s < NU; ++s) Ua[s] = Ub[s];
                    knot(a + 1, 0, Ub);
                }
            }
        };
        passes(
            [&]() __attribute__((always_inline)) -> T {
                double J = 0;
                v4 Js = zero;
                march(0, Tn, [&](const T *u, bool last) {
#pragma unroll
                    for (int q = 0; q < UT; ++q)
                        if (q == I.q)  // uniform
#pragma unroll
                            for (int s = 0; s < 4; ++s) {
                                const T e = I.Ug[s] - u[4 * q + s];
                                Js[s] += e * e;
                            }
                    if (last) {
#pragma unroll
                        for (int s = 0; s < 4; ++s) J += (double)I.Rw[s] * Js[s];
                        Js = zero;
                    }
                });
                J = over_rows(J);
                if (grp == 0) sR[w * 16 + col] = (T)J;
                lds_barrier();
                return total();
            },
            [&]() __attribute__((always_inline)) {
                // gA, gB: the current segment's sums for its two knots; carry: those
                // of the segment after it for the second one
                const d4 none = {0, 0, 0, 0};
                T r2[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) r2[s] = (T)2 * I.Rw[s];
                d4 gA = none, gB = none, carry = none;
                int a = p - 1, ka = seg_start(p - 1), par = 0;
                T Ua[4], Ub[4];  // own inputs of knots a and a + 1
                knot(a, 4 * I.q, Ua);
                knot(a + 1, 4 * I.q, Ub);
                for (int blk = G.nblk - 1; blk >= 0; --blk) {
                    const int k0 = G.full ? 0 : blk * G.S, k1 = G.full ? Tn : min(k0 + G.S, Tn);
                    if (!G.full) march(k0, k1 - 1, [](const T *, bool) {});
                    for (int k = k1 - 1; k >= k0; --k) {
                        const T c = sC[k];
                        v4 acc[4] = {zero, zero, zero, zero};
                        lds_barrier();
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            const v4 Lam = *tile(lam_at(par), t);
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int s = NT == 1 ? v : (v & 1) + 2 * (t & 1);
                                acc[s] = Mfma<T>::op(I.bT[4 * t + v], Lam[v], acc[s]);
                            }
                        }
                        par ^= 1;
                        const v4 bl = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const T u = ((T)1 - c) * Ua[s] + c * Ub[s];
                            const double g = r2[s] * (u - I.Ug[s]) + bl[s];
                            gA[s] += (double)((T)1 - c) * g;
                            gB[s] += (double)c * g;
                        }
                        if (k == ka) {  // segment a is done: knot a + 1 is complete
                            if (a < p - 1) knot_done(I, a + 1, carry + gB);
                            carry = gA;
                            if (a == 0) knot_done(I, 0, carry);
                            gA = gB = none;
                            --a;
                            ka = seg_start(a);
#pragma unroll
                            for (int s = 0; s < 4; ++s) Ub[s] = Ua[s];
                            knot(max(a, 0), 4 * I.q, Ua);
                        }
                    }
                }
            },
            w == NT);
        return;
    }

    // A state wavefront.  A operands by slot i (M-tile t =
    // (w + i) mod NT): rows of A_d and of A_d^T without the diagonal, which a
    // product adds last: discretized dynamics are close to the identity, and
    // every further term after the diagonal's rounds by the state's own size
    // (21-DoF chain, 100 steps, FP32: error of the gradient 9.7e-7 with the
    // diagonal in the sums, 4.8e-7 this way, 7.6e-7 in the per-candidate kernel).
    T aX[4 * NT], aT[4 * NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * w + arow, kk = 16 * ((w + i) % NT) + Mfma<T>::row(grp, v);
            const bool in = row < n && kk < n && row != kk;
            aX[4 * i + v] = in ? P.Ad[row * n + kk] : (T)0;
            aT[4 * i + v] = in ? P.Ad[kk * n + row] : (T)0;
        }
    // own rows: start state, goal, weights, box
    v4 X0, Xg, Q, Lo, Hi, Qb, Diag;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = 16 * w + Mfma<T>::row(grp, v);
        const bool in = row < n, bx = in && box;
        X0[v] = in ? x0[row] : (T)0;
        Diag[v] = in ? P.Ad[row * n + row] : (T)0;
        Xg[v] = in && P.xg ? P.xg[row] : (T)0;
        Q[v] = in ? P.q[row] : (T)0;
        sm[G.oQ + row] = in && P.qf ? P.qf[row] : (T)0;
        Lo[v] = bx ? P.xlo[row] : (T)-1;
        Hi[v] = bx ? P.xhi[row] : (T)1;
        Qb[v] = bx ? P.qb[row] : (T)0;
    }
    // M V over all M-tiles of a vector V, this wavefront's rows of the
    // matrix in `op` (by slot) and the diagonal, plus what `plus` adds to two of
    // the four partial sums: V's own tile from registers, the others from
    // `at`, where every wavefront has stored its own before the call.  The
    // barrier sits between the own slices, as in the M-split rollout, and
    // `shadow`, vector work of no use to this product, behind them.
    auto contract = [&](const T *op, v4 own, T *at, auto &&shadow, auto &&plus)
                        __attribute__((always_inline)) {
        // four partial sums, added pairwise: the rounding of the per-candidate
        // kernel's dot products (with two the gradient's error is 1.3 times
        // that, and the call 8 % faster)
        v4 acc[4] = {zero, zero, zero, zero};
        acc[0] = Mfma<T>::op(op[0], own[0], acc[0]);
        acc[1] = Mfma<T>::op(op[1], own[1], acc[1]);
        v4 o[NT];
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
#pragma unroll
        for (int i = 1; i < NT; ++i) o[i] = *tile(at, (w + i) % NT);
        constexpr int H = NT == 1 ? 2 : 0;
        acc[H] = Mfma<T>::op(op[2], own[2], acc[H]);
        acc[H + 1] = Mfma<T>::op(op[3], own[3], acc[H + 1]);
        shadow();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 1; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc[(v & 1) + 2 * (i & 1)] =
                    Mfma<T>::op(op[4 * i + v], o[i][v], acc[(v & 1) + 2 * (i & 1)]);
        v4 sum = (acc[0] + acc[1]) + plus(acc[2] + acc[3]);
#pragma unroll
        for (int v = 0; v < 4; ++v) sum[v] += Diag[v] * own[v];
        return sum;
    };
    // States x_{k0+1} .. x_{k1} from X = x_{k0}, which every wavefront has
    // stored at `at`; to(k): where x_k goes; each(x_k, k): called in the shadow of
    // the step that leaves x_k.
    auto march = [&](int k0, int k1, v4 X, T *at, auto &&to, auto &&each)
                     __attribute__((always_inline)) {
        for (int k = k0; k < k1; ++k) {
            v4 Bu;
            X = contract(
                aX, X, at,
                [&, X]() {
                    Bu = *tile(drive_at(k & 1), w);
                    each(X, k);
                },
                [](const v4 &sum) { return sum; });
            X += Bu;
            at = to(k + 1);
            *tile(at, w) = X;
        }
        return X;
    };
    // x_0 stays in its slot, which no pass overwrites; the terminal weights, of
    // use once per pass, in LDS too
    *tile(slot(0), w) = X0;
    auto terminal = [&](int v) { return sm[G.oQ + 16 * w + Mfma<T>::row(grp, v)]; };
    v4 XT;
    // cost of the knots in sU; leaves the states in LDS and x_T in XT
    auto forward = [&]() __attribute__((always_inline)) -> T {
        // sums over x_1 .. x_T: every step adds the state that it leaves, x_T
        // follows; x_0's terms are left out (selects: a branch would cut the
        // step), not subtracted, as their rounding would stay in the sums
        v4 S = zero, Pn = zero, Cn = zero;
        auto add = [&](const v4 &X, int k) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const T e = X[v] - Xg[v];
                S[v] = k > 0 ? S[v] + e * e : (T)0;
            }
            if (box) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    Pn[v] = k > 0 ? Pn[v] + box_pen(X[v], Lo[v], Hi[v]) : (T)0;
                    Cn[v] = k > 0 ? Cn[v] + box_out(X[v], Lo[v], Hi[v]) : (T)0;
                }
            }
        };
        const v4 Xs = *tile(slot(0), w);
        if (G.full) {
            T *at = slot(0);
            XT = march(
                0, Tn, Xs, at,
                // x_T is not read back: it goes into the ring of lambda, which is
                // idle here (not into a state's slot: other wavefronts may still
                // be reading the last step's, which for T = 1 is x_0's)
                [&](int k) -> T * {
                    at = k < Tn ? at + NT * 256 : lam_at(0);
                    return at;
                },
                add);
        } else {
            // the states between the blocks' first ones go through lambda's ring,
            // idle until the barrier that ends this pass
            T *ring = lam_at(0), *chk = slot(0);
            int q = 0;
            XT = march(
                0, Tn, Xs, chk,
                [&](int k) -> T * {
                    if (++q == G.S && k < Tn) {
                        q = 0;
                        chk += NT * 256;
                        return chk;
                    }
                    return ring + (k & 1) * (NT * 256);
                },
                add);
        }
        add(XT, Tn);
        double J = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double e = XT[v] - Xg[v];
            J += (double)Q[v] * S[v] + (double)terminal(v) * e * e;
            if (box) J += (double)Qb[v] * Pn[v];
        }
        if (box && P.sb) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * w + Mfma<T>::row(grp, v);
                J += row < n ? (double)P.sb[row] * Cn[v] : 0.0;
            }
        }
        J = over_rows(J);
        if (grp == 0) sR[w * 16 + col] = (T)J;
        lds_barrier();
        return total();
    };
    // dJ/dU of the knots, after forward()
    auto backward = [&]() __attribute__((always_inline)) {
        v4 L;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            L[v] = (T)2 * (Q[v] + terminal(v)) * (XT[v] - Xg[v]);
            if (box) L[v] += box_pen_grad(XT[v], Lo[v], Hi[v], Qb[v]);
        }
        int par = 0;
        for (int blk = G.nblk - 1; blk >= 0; --blk) {
            const int k0 = G.full ? 0 : blk * G.S, k1 = G.full ? Tn : min(k0 + G.S, Tn);
            T *seg = slot(G.full ? 0 : G.nblk);
            if (!G.full) {
                // x_{k0} .. x_{k1-1} into the block's slots
                const v4 X = *tile(slot(blk), w);
                *tile(seg, w) = X;
                march(k0, k1 - 1, X, slot(blk),
                      [&](int k) -> T * { return seg + (k - k0) * (NT * 256); },
                      [](const v4 &, int) {});
            }
            v4 X = *tile(seg + (k1 - 1 - k0) * (NT * 256), w);
            for (int k = k1 - 1; k >= k0; --k) {
                T *at = lam_at(par);
                par ^= 1;
                *tile(at, w) = L;
                if (k >= 1) {
                    v4 e, s = zero;
                    L = contract(
                        aT, L, at,
                        [&]() {
                            e = (T)2 * (X - Xg);
                            if (box) {
#pragma unroll
                                for (int v = 0; v < 4; ++v)
                                    s[v] = box_pen_grad(X[v], Lo[v], Hi[v], Qb[v]);
                            }
                            X = *tile(seg + (k > k0 ? k - 1 - k0 : 0) * (NT * 256), w);
                        },
                        [&](v4 sum) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) sum[v] += Q[v] * e[v];
                            return box ? sum + s : sum;
                        });
                } else {
                    lds_barrier();
                }
            }
        }
    };
    passes(forward, backward, false);
}

// Runs the call here if the tile's LDS fits; *taken tells.  All states are
// kept when they fit and the chip holds every tile at once that way;
// otherwise blocks of the length that needs the fewest slots.
template <typename T>
hipError_t launch_adjoint_linear_t(const ProbView<T> &P, const T *x0, const T *knots,
                                   int64_t ncand, int64_t ld, T *dJ, T *cost, int steps, T lr,
                                   T *knots_io, T *cost_io, hipStream_t s, bool *taken) {
    const int NT = (P.n + 15) / 16, UT = (P.m + 15) / 16;
    *taken = false;
    // the shapes instantiated below: no more input than state tiles, and no
    // shape whose registers spill to scratch (FP64 above 48 states or 32 inputs,
    // FP32 above 48 states with more than 32 inputs); the segment arithmetic is
    // in 32 bits
    if (NT > (sizeof(T) == 8 ? 3 : 4) || UT > NT || UT > (NT == 4 || sizeof(T) == 8 ? 2 : 3) ||
        (int64_t)P.Tn * P.p > (1 << 30))
        return hipSuccess;
    const int64_t tiles = (ncand + 15) / 16;
    auto bytes = [&](const LinAdjPlan &g) { return g.total * sizeof(T); };
    LinAdjPlan G = lin_adj_layout(NT, UT, P.Tn, P.p, steps > 0, P.Tn, true);
    const int64_t fit = bytes(G) <= MAX_GRAD_LDS ? (int64_t)(MAX_GRAD_LDS / bytes(G)) : 0;
    if (fit == 0 || tiles > 256 * fit) {
        int S = 1;
        while ((int64_t)S * S < P.Tn) ++S;
        const LinAdjPlan B = lin_adj_layout(NT, UT, P.Tn, P.p, steps > 0, S, false);
        if (bytes(B) <= MAX_GRAD_LDS) G = B;
    }
    if (bytes(G) > MAX_GRAD_LDS) return hipSuccess;
    // Few candidates: up to the number that the per-candidate kernel holds at
    // once (by its registers, 4, 2 or 1 workgroups per CU, and its LDS) it takes
    // the time of one, about 2 T + sqrt(T) steps.  A tile's steps are shorter in
    // FP32 up to 48 states, but it starts up longer and takes 3 T of them when its
    // states do not fit.  us per call, that kernel / here, 32 to 1024 candidates:
    //  FP32 n = 14, gradient: T = 10 13 / 14, T = 20 21 / 19, T = 100 75 / 61, in
    //   blocks T = 150 108 / 120; three Adam steps: T = 20 59 / 61, T = 35 94 / 89
    //  FP32 n = 28: T = 20 25 / 23, T = 50 49 / 43, in blocks T = 75 69 / 83;
    //   three Adam steps T = 20 70 / 74, T = 50 150 / 144, in blocks T = 75 218 / 272
    //  FP32 n = 42: T = 35 51 / 46, in blocks T = 50 68 / 83
    //  FP32 n = 60: T = 20 34 / 39; FP64 n = 14: T = 50 43 / 48, in blocks T = 75
    //   61 / 95; FP64 n = 28: T = 20 30 / 33, in blocks T = 50 62 / 96
    //  FP64 n = 42 (that kernel spills): T = 20 81 / 58
    //  a knot per step or two, FP32 n = 18, T = p = 50: 54 / 59
    // Above that number it takes a multiple of its time (FP32 n = 42, T = 100: 128
    // at 512 candidates, 254 at 768, 159 here).
    const size_t other = grad_smem_bytes(EMPC_LINEAR, P.n, P.m, P.Tn, P.p, sizeof(T));
    const int64_t by_regs = sizeof(T) == 4 ? (P.n <= 32 ? 4 : 2) : (P.n <= 16 ? 4 : P.n <= 32 ? 2 : 1);
    const int64_t held = 256 * std::min<int64_t>(by_regs, MAX_GRAD_LDS / other);
    const bool shorter = sizeof(T) == 8 ? NT > 2
                                        : NT < 4 && G.full && 3 * P.p <= P.Tn &&
                                              P.Tn >= (steps > 0 ? 28 : 16);
    if (ncand <= held && !shorter) return hipSuccess;
    *taken = true;
    auto go = [&](auto kernel) {
        if (bytes(G) > 65536) {
            const hipError_t e = hipFuncSetAttribute((const void *)kernel,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)bytes(G));
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(64 * (NT + UT)),
                           bytes(G), s, P, G, x0,
                           knots, ncand, ld, dJ, cost, steps, lr, knots_io, cost_io);
        return hipGetLastError();
    };
    switch (10 * NT + UT) {
        case 11: return go(adjoint_linear_kernel<T, 1, 1>);
        case 21: return go(adjoint_linear_kernel<T, 2, 1>);
        case 22: return go(adjoint_linear_kernel<T, 2, 2>);
        case 31: return go(adjoint_linear_kernel<T, 3, 1>);
        case 32: return go(adjoint_linear_kernel<T, 3, 2>);
        default: break;
    }
    if constexpr (sizeof(T) == 4) {
        if (NT == 3) return go(adjoint_linear_kernel<T, 3, 3>);
        if (UT == 1) return go(adjoint_linear_kernel<T, 4, 1>);
        return go(adjoint_linear_kernel<T, 4, 2>);
    }
    return hipErrorInvalidValue;  // not reached: excluded above
}

}  // namespace empc
