// Adjoint gradient and Adam refinement of the linear model on the matrix
// cores (gfx950), shared by the FP32 and FP64 translation units.
//
// A tile of 16 candidates runs on a workgroup of NT = ceil(n / 16)
// wavefronts, wavefront w owning state rows 16w .. 16w+15, in the accumulator
// layout and K order of the M-split rollout (rollout_linear.hpp).  The
// backward recursion lambda_k = 2 Q (x_k - g) + A^T lambda_{k+1} is the same
// contraction with A transposed, so the adjoint chains through the
// accumulators as the state does.  dJ/dU_j needs B^T lambda only through its
// knot-weighted sums: sum_k w_k(j) lambda_{k+1} is summed in registers and
// multiplied by B^T once per knot; the input weights' part is closed form in
// the sums of (1-c)^2, c (1-c) and c^2 over the knot segments.  The tile's
// knots sit in LDS, and so do the states of the forward pass: all of them
// when they fit (2 T dependent steps), else one per block of S steps, each
// block recomputed before it is walked backward (3 T steps).  Above one
// M-tile a further wavefront takes the input side (the input cost, the
// knots' products with B^T) while the state wavefronts go on: 43 -> 39 us.
//
// What bounds it is the chain of dependent steps (4 NT MFMAs in two chains, an
// LDS round trip and a barrier each), as in the M-split rollout: one
// wavefront pair per candidate took the same chain for a single candidate.
// 14-DoF chain, T = 50, p = 10, FP32, 4096 candidates: 238 us with a workgroup
// per candidate on the vector ALUs, 42 us here (65536: 3.2 ms and 0.55 ms); 64
// candidates with five Adam steps: 235 and 203 us.
#pragma once
#include <math.h>

#include <algorithm>

#include "internal.hpp"
#include "rollout_linear.hpp"

namespace empc {

// LDS plan (element counts) and the way the states are kept.
struct LinAdjPlan {
    int full;          // every state kept
    int S, nblk;       // steps per block and blocks (full: one block)
    size_t oX, oL, oK, oR, oS, oU, oM1, oM2, oG, total;
};
inline LinAdjPlan lin_adj_layout(int NT, int NU, int T, int p, bool refine, int S, bool full) {
    LinAdjPlan g;
    g.full = full;
    g.S = S;
    g.nblk = full ? 1 : (T + S - 1) / S;
    const size_t slot = (size_t)NT * 256, kn = (size_t)p * NU * 64;
    size_t o = 0;
    // full: x_0 .. x_{T-1}; else the blocks' first states, one block, a ring of two
    g.oX = o; o += slot * (full ? (size_t)T : (size_t)g.nblk + S + 2);
    g.oL = o; o += 2 * slot;
    g.oK = o; o += 3 * slot;
    g.oU = o; o += kn;
    g.oM1 = o; o += refine ? kn : 0;
    g.oM2 = o; o += refine ? kn : 0;
    g.oG = o; o += refine ? kn : 0;
    g.oS = o; o += (size_t)3 * p;
    g.oR = o; o += (size_t)(NT + 1) * 16;
    g.total = o;
    return g;
}

// wavefronts of a tile: the NT state wavefronts, and above one of them a
// further one for the inputs
template <int NT>
constexpr int ADJ_WAVES = NT > 1 ? NT + 1 : 1;

template <typename T, int NT, int UT>
__global__ __launch_bounds__(64 * ADJ_WAVES<NT>) void adjoint_linear_kernel(
    ProbView<T> P, LinAdjPlan G, const T *__restrict__ x0, const T *__restrict__ knots,
    int64_t ncand, int64_t ld, T *__restrict__ dJ, T *__restrict__ cost, int steps, T lr,
    T *__restrict__ knots_io, T *__restrict__ cost_io) {
    typedef typename Mfma<T>::v4 v4;
    constexpr int NU = 4 * UT, KN = NU * 64;  // input slices; elements of one knot
    extern __shared__ __align__(32) unsigned char adj_smem[];
    T *sm = (T *)adj_smem;
    T *sU = sm + G.oU, *sS = sm + G.oS, *sR = sm + G.oR;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int64_t cand = xcd_swizzle(blockIdx.x, gridDim.x) * 16 + col;
    const bool valid = cand < ncand, refine = steps > 0;
    const int n = P.n, m = P.m, p = P.p, Tn = P.Tn;
    const bool box = P.qb != nullptr;  // uniform
    const int arow = Mfma<T>::mstate(col);

    constexpr int NW = ADJ_WAVES<NT>;
    const bool inputs = w == NW - 1;  // runs the input side (with one wavefront: everything)
    // the tile's knots, [knot][slice][lane]: lane (grp, col) of slice s holds
    // input 4 s + grp of candidate col (past m or the candidates: a value
    // that is never stored and meets zero weights); the first loads are in
    // flight while the operands are loaded
    const T *src = refine ? knots_io : knots;
    const int64_t cand_c = valid ? cand : ncand - 1;
    constexpr int LB = 16;
    T first[LB];
    auto load_knots = [&](int e0) {
#pragma unroll
        for (int b = 0; b < LB; ++b) {
            const int e = min(e0 + b * NW, p * NU - 1), i = 4 * (e % NU) + grp;
            first[b] = src[(int64_t)((e / NU) * m + min(i, m - 1)) * ld + cand_c];
        }
    };
    auto store_knots = [&](int e0) {
#pragma unroll
        for (int b = 0; b < LB; ++b) {
            const int e = e0 + b * NW;
            if (e < p * NU) sU[e * 64 + lane] = 4 * (e % NU) + grp < m ? first[b] : (T)0;
        }
    };
    load_knots(w);

    // A operands of the state wavefronts by slot i (M-tile t = (w + i) mod
    // NT): rows of A_d and of A_d^T; B_d's rows by input slice
    T aX[4 * NT], aT[4 * NT], aU[NU];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * w + arow, kk = 16 * ((w + i) % NT) + Mfma<T>::row(grp, v);
            const bool in = row < n && kk < n;
            aX[4 * i + v] = in ? P.Ad[row * n + kk] : (T)0;
            aT[4 * i + v] = in ? P.Ad[kk * n + row] : (T)0;
        }
#pragma unroll
    for (int s = 0; s < NU; ++s) {
        const int row = 16 * w + arow, j = 4 * s + grp;
        aU[s] = row < n && j < m ? P.Bd[row * m + j] : (T)0;
    }
    // own rows: start state, disturbance, goal, weights, box
    v4 X0, Wd, Xg, Q, Qf, Lo, Hi, Qb, Sb;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = 16 * w + Mfma<T>::row(grp, v);
        const bool in = row < n, bx = in && box;
        X0[v] = in ? x0[row] : (T)0;
        Wd[v] = in && P.wd ? P.wd[row] : (T)0;
        Xg[v] = in && P.xg ? P.xg[row] : (T)0;
        Q[v] = in ? P.q[row] : (T)0;
        Qf[v] = in && P.qf ? P.qf[row] : (T)0;
        Lo[v] = bx ? P.xlo[row] : (T)-1;
        Hi[v] = bx ? P.xhi[row] : (T)1;
        Qb[v] = bx ? P.qb[row] : (T)0;
        Sb[v] = bx && P.sb ? P.sb[row] : (T)0;
    }
    // the input side: rows of B_d^T of output tile u by M-tile, weights and
    // goals (tile u, register s: input 16 u + 4 s + grp)
    T bT[UT][4 * NT], Rw[UT][4], Ug[UT][4];
#pragma unroll
    for (int u = 0; u < UT; ++u) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * u + arow, kk = 16 * i + Mfma<T>::row(grp, v);
                bT[u][4 * i + v] = inputs && row < m && kk < n ? P.Bd[kk * m + row] : (T)0;
            }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int i = 16 * u + 4 * s + grp;
            Rw[u][s] = i < m ? P.r[i] : (T)0;
            Ug[u][s] = i < m && P.ug ? P.ug[i] : (T)0;
        }
    }
    store_knots(w);
    for (int e0 = w + LB * NW; e0 < p * NU; e0 += LB * NW) {
        load_knots(e0);
        store_knots(e0);
    }
    if (refine)
        for (int e = threadIdx.x; e < p * KN; e += 64 * NW) sm[G.oM1 + e] = sm[G.oM2 + e] = 0;
    const T inv_den = Tn > 1 ? (T)1 / (T)(Tn - 1) : (T)0;
    // first step of segment a (steps with idx1 = a)
    auto seg_start = [&](int a) {
        return p == 1 ? (a == 0 ? 0 : Tn) : a >= p ? Tn : (a * (Tn - 1) + p - 2) / (p - 1);
    };
    auto weight = [&](int k, int a) {
        return (T)(k * (p - 1) - a * (Tn - 1)) * inv_den;  // 0 for one knot or one step
    };
    // sums of (1-c)^2, c (1-c), c^2 over each segment
    for (int a = threadIdx.x; a < p; a += 64 * NW) {
        T s00 = 0, s01 = 0, s11 = 0;
        for (int k = seg_start(a); k < seg_start(a + 1); ++k) {
            const T c = weight(k, a), d = (T)1 - c;
            s00 += d * d;
            s01 += c * d;
            s11 += c * c;
        }
        sS[3 * a] = s00;
        sS[3 * a + 1] = s01;
        sS[3 * a + 2] = s11;
    }
    auto tile = [&](T *slot, int t) { return reinterpret_cast<v4 *>(slot) + t * 64 + lane; };
    auto slot = [&](int k) { return sm + G.oX + (size_t)k * NT * 256; };
    // start + M V over all M-tiles of a vector V, this wavefront's rows of the
    // matrix in `op` (by slot): V's own tile from registers, the others from
    // `at`, where every wavefront has stored its own before the call.  The
    // barrier sits between the own slices, as in the M-split rollout, and
    // `shadow`, vector work of no use to this step, behind them.
    auto contract = [&](const T *op, v4 own, T *at, v4 start, auto &&shadow)
                        __attribute__((always_inline)) {
        // four partial sums, added pairwise: the rounding of the per-candidate
        // kernel's dot products (with two the gradient's error is 1.3 times
        // that, and the call 8 % faster)
        v4 acc[4] = {start, v4{0, 0, 0, 0}, v4{0, 0, 0, 0}, v4{0, 0, 0, 0}};
        acc[0] = Mfma<T>::op(op[0], own[0], acc[0]);
        acc[1] = Mfma<T>::op(op[1], own[1], acc[1]);
        v4 o[NT];
        if (NT > 1) {
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();
#pragma unroll
            for (int i = 1; i < NT; ++i) o[i] = *tile(at, (w + i) % NT);
        }
        constexpr int H = NT == 1 ? 2 : 0;
        acc[H] = Mfma<T>::op(op[2], own[2], acc[H]);
        acc[H + 1] = Mfma<T>::op(op[3], own[3], acc[H + 1]);
        shadow();
        if (NT > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 1; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc[(v & 1) + 2 * (i & 1)] =
                    Mfma<T>::op(op[4 * i + v], o[i][v], acc[(v & 1) + 2 * (i & 1)]);
        return (acc[0] + acc[1]) + (acc[2] + acc[3]);
    };
    // own rows of V = B_d U + w_d for knot j
    auto response = [&](int j) __attribute__((always_inline)) {
        const T *u = sU + (size_t)(j < p ? j : p - 1) * KN + lane;
        v4 V[2] = {Wd, v4{0, 0, 0, 0}};
#pragma unroll
        for (int s = 0; s < NU; ++s) V[s & 1] = Mfma<T>::op(aU[s], u[64 * s], V[s & 1]);
        return V[0] + V[1];
    };
    // states x_{k0+1} .. x_{k1} from X = x_{k0}, which every wavefront has
    // stored at `at`; to(k): where x_k goes; each(x_k, k): called in the shadow
    // of the step that leaves x_k
    auto march = [&](int k0, int k1, v4 X, T *at, auto &&to, auto &&each)
                     __attribute__((always_inline)) {
        int a = p == 1 || Tn == 1 ? 0 : k0 * (p - 1) / (Tn - 1);
        v4 Va = response(a), Vb = response(a + 1);
        for (int k = k0; k < k1; ++a) {
            const int ke = min(seg_start(a + 1), k1);
            const v4 dV = Vb - Va;
            v4 start = Va + weight(k, a) * dV;
            for (; k < ke; ++k) {
                const v4 s0 = start;
                X = contract(aX, X, at, s0, [&, X]() {
                    each(X, k);
                    start = Va + weight(k + 1, a) * dV;
                });
                at = to(k + 1);
                *tile(at, w) = X;
            }
            Va = Vb;
            if (k < k1) Vb = response(a + 2);
        }
        return X;
    };
    // input side of the cost: each segment's part in closed form
    auto input_cost = [&]() __attribute__((always_inline)) {
        T J = 0;
        for (int a = 0; a < p; ++a) {
            const T *u0 = sU + (size_t)a * KN + lane, *u1 = a + 1 < p ? u0 + KN : u0;
            const T s00 = sS[3 * a], s01 = sS[3 * a + 1], s11 = sS[3 * a + 2];
#pragma unroll
            for (int u = 0; u < UT; ++u)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const T e0 = u0[256 * u + 64 * s] - Ug[u][s];
                    const T e1 = u1[256 * u + 64 * s] - Ug[u][s];
                    J += Rw[u][s] * (s00 * e0 * e0 + (T)2 * s01 * e0 * e1 + s11 * e1 * e1);
                }
        }
        return J;
    };
    // dJ/dU_j from the weighted sum of lambda that the state wavefronts left
    // at `at`: to dJ, or to G when refining
    auto knot_grad = [&](int j, T *at) __attribute__((always_inline)) {
        const T cc = sS[3 * j] + (j > 0 ? sS[3 * j - 1] : (T)0);
        const T cn = j < p - 1 ? sS[3 * j + 1] : (T)0, cp = j > 0 ? sS[3 * j - 2] : (T)0;
#pragma unroll
        for (int u = 0; u < UT; ++u) {
            const T *uj = sU + (size_t)j * KN + 256 * u + lane;
            const T *un = j < p - 1 ? uj + KN : uj, *up = j > 0 ? uj - KN : uj;
            v4 acc[2] = {v4{0, 0, 0, 0}, v4{0, 0, 0, 0}};
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const v4 o = *tile(at, t);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[v & 1] = Mfma<T>::op(bT[u][4 * t + v], o[v], acc[v & 1]);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const T g = acc[0][s] + acc[1][s] +
                            (T)2 * Rw[u][s] *
                                (cc * (uj[64 * s] - Ug[u][s]) + cn * (un[64 * s] - Ug[u][s]) +
                                 cp * (up[64 * s] - Ug[u][s]));
                const int i = 16 * u + 4 * s + grp;
                if (refine)
                    sm[G.oG + (size_t)j * KN + 256 * u + 64 * s + lane] = g;
                else if (i < m && valid)
                    dJ[(int64_t)(j * m + i) * ld + cand] = g;
            }
        }
    };
    auto lam_at = [&](int i) { return sm + G.oK + i * (NT * 256); };  // ring of three
    auto next3 = [](int i) { return i == 2 ? 0 : i + 1; };
    // The input wavefront (NT > 1) passes the state wavefronts' barriers: one
    // per step of a march, one per backward step, one after the last
    auto forward_inputs = [&]() __attribute__((always_inline)) -> T {
        for (int k = 0; k < Tn; ++k) {
            if (k == 0) {
                T J = input_cost();
                J += __shfl_xor(J, 16, 64);
                J += __shfl_xor(J, 32, 64);
                if (grp == 0) sR[NT * 16 + col] = J;
            }
            lds_barrier();
        }
        lds_barrier();
        T J = sR[col];
#pragma unroll
        for (int t = 1; t <= NT; ++t) J += sR[t * 16 + col];
        return J;
    };
    auto backward_inputs = [&]() __attribute__((always_inline)) {
        int a = p - 1, ka = seg_start(p - 1), buf = 0, due = -1;
        for (int blk = G.nblk - 1; blk >= 0; --blk) {
            const int k0 = G.full ? 0 : blk * G.S, k1 = G.full ? Tn : min(k0 + G.S, Tn);
            if (!G.full)
                for (int k = k0; k < k1 - 1; ++k) lds_barrier();
            for (int k = k1 - 1; k >= k0; --k) {
                lds_barrier();
                if (due >= 0) {  // published before this barrier
                    knot_grad(due, lam_at(buf));
                    buf = next3(buf);
                    due = -1;
                }
                if (k == ka) {
                    due = a < p - 1 ? a + 1 : -1;
                    --a;
                    ka = seg_start(a);
                }
            }
        }
        lds_barrier();
        if (due >= 0) {
            knot_grad(due, lam_at(buf));
            buf = next3(buf);
        }
        knot_grad(0, lam_at(buf));
    };
    // cost of the knots in sU; leaves the states in LDS and x_T in XT
    v4 XT = X0;
    auto forward = [&]() __attribute__((always_inline)) -> T {
        // sums over x_1 .. x_T: every step adds the state that it leaves, x_T
        // follows; x_0's terms are left out (selects: a branch would cut the
        // step), not subtracted, as their rounding would stay in the sums
        v4 S = {0, 0, 0, 0}, Pn = {0, 0, 0, 0}, Cn = {0, 0, 0, 0};
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
        *tile(slot(0), w) = X0;
        if (G.full) {
            T *at = slot(0);
            XT = march(
                0, Tn, X0, at,
                // x_T is not read back: it goes into the ring of lambda, which is
                // idle here (not into a state's slot: other wavefronts may still
                // be reading the last step's, which for T = 1 is x_0's)
                [&](int k) -> T * {
                    at = k < Tn ? at + NT * 256 : sm + G.oL;
                    return at;
                },
                add);
        } else {
            T *ring = slot(G.nblk + G.S), *chk = slot(0);
            int q = 0;
            XT = march(
                0, Tn, X0, chk,
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
        T J = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const T e = XT[v] - Xg[v];
            J += Q[v] * S[v] + Qf[v] * e * e;
            if (box) J += Qb[v] * Pn[v] + Sb[v] * Cn[v];
        }
        if (NT == 1) J += input_cost();
        J += __shfl_xor(J, 16, 64);
        J += __shfl_xor(J, 32, 64);
        if (NT == 1) return J;
        if (grp == 0) sR[w * 16 + col] = J;
        lds_barrier();
        J = sR[col];
#pragma unroll
        for (int t = 1; t <= NT; ++t) J += sR[t * 16 + col];
        return J;
    };
    // dJ/dU of the knots, after forward(): to dJ, or to G when refining
    auto backward = [&]() __attribute__((always_inline)) {
        v4 L, gA = {0, 0, 0, 0}, gB = {0, 0, 0, 0}, carry = {0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            L[v] = (T)2 * (Q[v] + Qf[v]) * (XT[v] - Xg[v]);
            if (box) L[v] += box_pen_grad(XT[v], Lo[v], Hi[v], Qb[v]);
        }
        int par = 0, buf = 0;
        // knot j's weighted sum of lambda is complete: the input wavefront
        // takes it after the next barrier
        auto flush = [&](int j, const v4 &Lam) {
            *tile(lam_at(buf), w) = Lam;
            if (NT == 1) knot_grad(j, lam_at(buf));
            buf = next3(buf);
        };
        int a = p - 1, ka = seg_start(p - 1);
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
                const T c = weight(k, a);
                auto sums = [&, L]() {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        gA[v] += ((T)1 - c) * L[v];
                        gB[v] += c * L[v];
                    }
                };
                if (k >= 1) {
                    T *at = sm + G.oL + par * (NT * 256);
                    par ^= 1;
                    if (NT > 1) *tile(at, w) = L;
                    v4 s;
                    L = contract(aT, L, at, v4{0, 0, 0, 0}, [&]() {
                        sums();
#pragma unroll
                        for (int v = 0; v < 4; ++v) s[v] = (T)2 * Q[v] * (X[v] - Xg[v]);
                        if (box) {
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                s[v] += box_pen_grad(X[v], Lo[v], Hi[v], Qb[v]);
                        }
                        X = *tile(seg + (k > k0 ? k - 1 - k0 : 0) * (NT * 256), w);
                    });
                    L += s;
                } else {
                    if (NT > 1) lds_barrier();
                    sums();
                }
                if (k == ka) {  // segment a is done: knot a + 1 is complete
                    if (a < p - 1) flush(a + 1, carry + gB);
                    carry = gA;
                    gA = gB = v4{0, 0, 0, 0};
                    --a;
                    ka = seg_start(a);
                }
            }
        }
        flush(0, carry);
        if (NT > 1) lds_barrier();
    };

    auto run_forward = [&]() __attribute__((always_inline)) {
        return NT > 1 && inputs ? forward_inputs() : forward();
    };
    auto run_backward = [&]() __attribute__((always_inline)) {
        if (NT > 1 && inputs)
            backward_inputs();
        else
            backward();
    };
    lds_barrier();  // knots, sums
    if (!refine) {
        const T J = run_forward();
        if (cost && inputs && grp == 0 && valid) cost[cand] = J;
        run_backward();
        return;
    }
    // Adam (Kingma & Ba 2015), bias-corrected, clamp after each update
    const T b1 = (T)0.9, b2 = (T)0.999, eps = (T)1e-8;
    T b1t = 1, b2t = 1, J0 = 0;
    for (int t = 1; t <= steps; ++t) {
        const T Jt = run_forward();
        if (t == 1) J0 = Jt;
        run_backward();
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
    const T Jn = run_forward();
    if (valid && Jn < J0) {
        for (int e = w; e < p * NU; e += NW) {
            const int i = 4 * (e % NU) + grp;
            if (i < m) knots_io[(int64_t)((e / NU) * m + i) * ld + cand] = sU[e * 64 + lane];
        }
        if (inputs && grp == 0) cost_io[cand] = Jn;
    }
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
    // the shapes instantiated below (no more input than state tiles, and no
    // shape whose registers spill to scratch: FP64 above 48 states, FP32
    // above 48 with more than 32 inputs); the segment arithmetic is in 32 bits
    if (NT > (sizeof(T) == 8 ? 3 : 4) || UT > NT || UT > (NT == 4 ? 2 : 3) ||
        (int64_t)P.Tn * P.p > (1 << 30))
        return hipSuccess;
    // A tile's step takes 4 NT MFMAs whatever the number of candidates; the
    // per-candidate kernel holds 1024 (n <= 16) or 512 candidates at once and
    // up to there takes the time of one.  With few candidates it stays the
    // faster one where the MFMA chain is long (50 steps, us per call, that
    // kernel / here): FP32 n = 28 49 / 35, n = 42 68 / 64, n = 60 69 / 79 at
    // 64 candidates and 142 / 80 at 1024; FP64 n = 14 42 / 43 at 64 and
    // 128 / 44 at 2048, five Adam steps on 64 142 / 191, n = 28 61 / 75 at 64
    // and 124 / 77 at 1024.
    if ((sizeof(T) == 8 || NT == 4) && ncand <= (NT == 1 ? 1024 : 512)) return hipSuccess;
    const int64_t tiles = (ncand + 15) / 16;
    auto bytes = [&](const LinAdjPlan &g) { return g.total * sizeof(T); };
    LinAdjPlan G = lin_adj_layout(NT, 4 * UT, P.Tn, P.p, steps > 0, P.Tn, true);
    const int64_t fit = bytes(G) <= MAX_GRAD_LDS ? (int64_t)(MAX_GRAD_LDS / bytes(G)) : 0;
    if (fit == 0 || tiles > 256 * fit) {
        int S = 1;
        while ((int64_t)S * S < P.Tn) ++S;
        const LinAdjPlan B = lin_adj_layout(NT, 4 * UT, P.Tn, P.p, steps > 0, S, false);
        if (bytes(B) <= MAX_GRAD_LDS) G = B;
    }
    if (bytes(G) > MAX_GRAD_LDS) return hipSuccess;
    *taken = true;
    auto go = [&](auto kernel) {
        if (bytes(G) > 65536) {
            const hipError_t e = hipFuncSetAttribute((const void *)kernel,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)bytes(G));
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(64 * (NT > 1 ? NT + 1 : 1)),
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
        case 33: return go(adjoint_linear_kernel<T, 3, 3>);
        default: break;
    }
    if constexpr (sizeof(T) == 4) {
        if (UT == 1) return go(adjoint_linear_kernel<T, 4, 1>);
        return go(adjoint_linear_kernel<T, 4, 2>);
    }
    return hipErrorInvalidValue;  // not reached: excluded above
}

}  // namespace empc
