// Parameterized small-matrix convex MPC on the GPU (gfx950): the paper's
// other method (Sec. IV-B small-matrix formulation, parameterized as in
// Sec. IV-E), for linear problems.  With z the knot vector, the states
// x_1..x_T = S z + v and the cost of eq. 3 is J(z) = z^T P z + 2 q^T z + c;
// the knot bounds make the MPC a box-constrained QP.
//  - qp_traj_kernel: S and v.  One workgroup per column: the response of
//    unit knot j from rest (column j of S, built step by step as the paper
//    describes, each row the previous one times A_d plus B_d in the knot's
//    proportions), and one workgroup for the free response v from x0 with
//    w_d; one thread per state row with its row of A_d in registers, the
//    state exchanged through LDS each step (the paper's own
//    thread-per-state layout: the work is tiny, a step is one chain of n
//    dependent multiply-adds).
//  - qp_form_kernel: P = S^T Qb S + Phi^T Rb Phi in 16 x 16 output tiles on
//    the FP64 matrix cores, the input part in closed form from the knot
//    weights, and q and c.
//  - qp_box_small_kernel / qp_box_kernel: the box QP by the projected Newton
//    method (Bertsekas 1982): Newton steps of the quadratic restricted to
//    the variables off their bounds (Cholesky solves), an Armijo search along
//    the projection arc; one workgroup, the factor in LDS up to BOX_MAX_PM
//    knot parameters and in global memory above.
// A 16x16x4 MFMA adds its four products in ascending order, each a fused
// multiply-add (compared bit for bit with fma chains, FP64 and FP32), so the
// matrix-core forms round as the element-wise loops that they replaced and
// the iterates, and with them the iteration counts, are the same.
// Every step computes in FP64; inputs and outputs are in the problem dtype.
#include <hip/hip_runtime.h>
#include <math.h>

#include "internal.hpp"

namespace empc {

namespace {

constexpr int QP_THREADS = 1024;
constexpr int QP_MAX_PM = 1024;    // one knot parameter per QP thread

// weight of knot a at step k (u_k = (1-c) U_idx1 + c U_idx2)
__device__ inline double knot_weight(int T, int p, int k, int a) {
    const Knot s = knot_at(T, p, k);
    const double c = (double)s.rem / (double)s.den;
    return (a == s.a ? 1.0 - c : 0.0) + (a == s.b ? c : 0.0);
}

// first and last step whose inputs the knots a and a' both touch (lo > hi:
// none); the weights of every other step are zero for one of them
__device__ inline void knot_support(int T, int p, int a, int a2, int *lo, int *hi) {
    *lo = 0;
    *hi = T - 1;
    if (p == 1 || T == 1) return;
    const int l = (a > a2 ? a : a2) - 1, h = (a < a2 ? a : a2) + 1;
    if (h < l) {
        *hi = -1;
        return;
    }
    if (l > 0) *lo = (int)((int64_t)l * (T - 1) / (p - 1));
    const int64_t e = ((int64_t)h * (T - 1) + p - 2) / (p - 1);
    if (e < T - 1) *hi = (int)e;
}

// f(weight of knot a, weight of knot a2) for the steps that both touch, in
// ascending order (knot_weight's values, one division per step)
template <typename F>
__device__ inline void for_shared_steps(int T, int p, int a, int a2, F &&f) {
    int lo, hi;
    knot_support(T, p, a, a2, &lo, &hi);
    if (hi < lo) return;
    Knot s = knot_at(T, p, lo);
    for (int k = lo; k <= hi; ++k) {
        const double c = (double)s.rem / (double)s.den;
        f((a == s.a ? 1.0 - c : 0.0) + (a == s.b ? c : 0.0),
          (a2 == s.a ? 1.0 - c : 0.0) + (a2 == s.b ? c : 0.0));
        s.rem += p - 1;
        if (s.rem >= s.den && T > 1) {
            s.rem -= s.den;
            ++s.a;
            s.b = s.a + 1 < p ? s.a + 1 : p - 1;
        }
    }
}

// Columns of S ([T n][pm]) and the free response.
// NR >= n: length of the register row of A_d; THR threads, one per state row.
// The knot weights of 64 steps at a time are tabulated, so that the step
// holds no division.  14-DoF chain, 50 steps: 47 us with A_d read from memory
// in every step, 18 us now.
constexpr int TRAJ_CHUNK = 64;
template <typename T, int NR, int THR>
__global__ __launch_bounds__(THR) void qp_traj_kernel(ProbView<T> P, const T *__restrict__ x0,
                                                      double *__restrict__ S,
                                                      double *__restrict__ v) {
    __shared__ __align__(16) double x[2][NR];
    __shared__ double wk[TRAJ_CHUNK];
    typedef double v2 __attribute__((ext_vector_type(2)));
    const int n = P.n, m = P.m, pm = P.p * P.m, r = threadIdx.x;
    const int j = blockIdx.x;  // column; j == pm: the free response
    const bool free_resp = j == pm;
    const int aj = free_resp ? 0 : j / m, ij = free_resp ? 0 : j % m;
    const bool in = r < n;
    double a[NR];
#pragma unroll
    for (int c = 0; c < NR; ++c) a[c] = in && c < n ? (double)P.Ad[r * n + c] : 0.0;
    const double bd = in ? (free_resp ? (P.wd ? (double)P.wd[r] : 0.0) : (double)P.Bd[r * m + ij])
                         : 0.0;
    if (r < NR) {
        x[0][r] = free_resp && in ? (double)x0[r] : 0.0;
        x[1][r] = 0.0;
    }
    double *out = free_resp ? v + r : S + (int64_t)r * pm + j;
    const int64_t step = free_resp ? n : (int64_t)n * pm;
    for (int k0 = 0; k0 < P.Tn; k0 += TRAJ_CHUNK) {
        __syncthreads();
        if (r < TRAJ_CHUNK && k0 + r < P.Tn)
            wk[r] = free_resp ? 1.0 : knot_weight(P.Tn, P.p, k0 + r, aj);
        __syncthreads();
        const int ke = P.Tn - k0 < TRAJ_CHUNK ? P.Tn - k0 : TRAJ_CHUNK;
        for (int kk = 0; kk < ke; ++kk) {
            const int k = k0 + kk;
            const double *xc = x[k & 1];
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < NR; c += 2) {
                const v2 xv = *reinterpret_cast<const v2 *>(xc + c);
                s += a[c] * xv.x;
                s += a[c + 1] * xv.y;
            }
            s += bd * wk[kk];
            if (in) {
                x[(k + 1) & 1][r] = s;
                out[k * step] = s;
            }
            __syncthreads();
        }
    }
}

// P, q and c from S and v.  Blocks below tiles^2: one 16 x 16 tile of P;
// wavefront z sums slice z of the stacked state rows K = k n + r, weight q_r
// (+ qf_r at x_T), on the FP64 matrix cores (w_K S[K][i] S[K][j]), the slices
// are added in order, then the input part sum_k w_k(knot of i) w_k(knot of j)
// r_input on matching inputs.  The next `tiles` blocks: q, 16 columns each, and
// the last one c: sums over the stacked rows in 256 strided parts, reduced in
// LDS in halves.  Both read S 16 columns wide, a cache line per row (column
// by column, 16 rows to a load, the kernel took 25 us).
// 14-DoF chain (140 parameters, 1400 rows): 15 + 25 + 5 us in three launches
// (VALU tiles; the slice sum recomputed every knot weight of the horizon for
// each element), 16 us in this one.
constexpr int GRAM_SPLIT = 8;
constexpr int FORM_THREADS = 64 * GRAM_SPLIT;
constexpr int FORM_MAX_N = 80;
typedef double v4d __attribute__((ext_vector_type(4)));
template <typename T>
__global__ __launch_bounds__(FORM_THREADS) void qp_form_kernel(
    ProbView<T> P, const double *__restrict__ S, const double *__restrict__ v, int tiles,
    T *__restrict__ Pout, T *__restrict__ qout, T *__restrict__ cout) {
    constexpr int PARTS = 256;  // of the sums for q and c
    __shared__ double part[16 * PARTS];
    __shared__ double wq[2][FORM_MAX_N];  // stage weights, and those of x_T
    static_assert(GRAM_SPLIT * 256 <= 16 * PARTS, "slices fit");
    const int pm = P.p * P.m, n = P.n, K = P.Tn * n, m = P.m, tid = threadIdx.x;
    if (tid < n) {
        const double q = (double)P.q[tid];
        wq[0][tid] = q;
        wq[1][tid] = P.qf ? q + (double)P.qf[tid] : q;
    }
    __syncthreads();
    if ((int)blockIdx.x < tiles * tiles) {
        const int i0 = (int)(blockIdx.x / tiles) * 16, j0 = (int)(blockIdx.x % tiles) * 16;
        const int lane = tid & 63, z = tid >> 6, g = lane >> 4, c = lane & 15;
        const int kb = (int)((int64_t)K * z / GRAM_SPLIT);
        const int ke = (int)((int64_t)K * (z + 1) / GRAM_SPLIT);
        const double *Si = S + min(i0 + c, pm - 1), *Sj = S + min(j0 + c, pm - 1);
        v4d acc = {0, 0, 0, 0};
        int kr = kb + g, k = kr / n, r = kr % n;
        // MFMAs per batch of loads in flight.  A slice ends within a batch, whose
        // rest multiplies zeros: 8, 12, 16, 22 per batch, us: 400 rows of 40
        // parameters 8.4, 9.5, 8.6, 9.9; 1400 of 140 16.8, 16.3, 16.3, 15.7;
        // 1500 of 150 16.8, 16.6, 16.3, 19.6.
        constexpr int U = 8;
        for (int k0 = kb; k0 < ke; k0 += 4 * U) {
            double a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t kk = (int64_t)min(kr + 4 * u, ke - 1) * pm;
                a[u] = Si[kk];
                b[u] = Sj[kk];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // past the slice: the weight and the second factor are zero
                const bool ok = kr + 4 * u < ke;
                const double w = wq[k == P.Tn - 1 ? 1 : 0][r];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ok ? w * a[u] : 0.0, ok ? b[u] : 0.0,
                                                           acc, 0, 0, 0);
                if (n >= 4) {  // uniform
                    const bool wrap = r + 4 >= n;
                    r += wrap ? 4 - n : 4;
                    k += wrap ? 1 : 0;
                } else {
                    k = (kr + 4 * u + 4) / n;
                    r = (kr + 4 * u + 4) % n;
                }
            }
            kr += 4 * U;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) part[256 * z + (g + 4 * q) * 16 + c] = acc[q];
        __syncthreads();
        const int i = i0 + tid / 16, j = j0 + tid % 16;
        if (tid < 256 && i < pm && j < pm) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < GRAM_SPLIT; ++q) s += part[256 * q + tid];
            if (i % m == j % m) {
                double t = 0.0;
                for_shared_steps(P.Tn, P.p, i / m, j / m, [&](double wi, double wj) { t += wi * wj; });
                s += t * (double)P.r[i % m];
            }
            Pout[(int64_t)i * pm + j] = (T)s;
        }
        return;
    }
    // part t sums the rows t, t + 256, ..; thread: parts tid / 16 + 32 u of
    // column tid mod 16 (the block of c: column 0 only)
    const int blk = (int)blockIdx.x - tiles * tiles;
    const bool of_c = blk == tiles;
    const int c = tid & 15, i = of_c ? 0 : 16 * blk + c;
    constexpr int U = 16 * PARTS / FORM_THREADS;  // parts per thread, their loads in flight together
    const int dk = PARTS / n, dr = PARTS % n, t0 = tid >> 4;
    const bool on = of_c ? c == 0 : i < pm;
    const double *Sc = S + min(i, pm - 1);
    double s[U];
    int k[U], r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = t0 + FORM_THREADS / 16 * u;
        s[u] = 0.0;
        k[u] = t / n;
        r[u] = t % n;
    }
    for (int kr0 = t0; kr0 < K; kr0 += PARTS) {
        double x[U], vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kr = min(kr0 + FORM_THREADS / 16 * u, K - 1);
            x[u] = of_c ? 0.0 : Sc[(int64_t)kr * pm];
            vv[u] = v[kr];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kr0 + FORM_THREADS / 16 * u < K) {
                const double w = wq[k[u] == P.Tn - 1 ? 1 : 0][r[u]];
                const double e = vv[u] - (P.xg ? (double)P.xg[r[u]] : 0.0);
                if (of_c)
                    s[u] += w * e * e;
                else
                    s[u] += x[u] * w * e;
            }
            k[u] += dk;
            r[u] += dr;
            if (r[u] >= n) {
                r[u] -= n;
                ++k[u];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = t0 + FORM_THREADS / 16 * u;
        if (P.ug && of_c)
            for (int ii = t; ii < m; ii += PARTS)
                s[u] += (double)P.Tn * (double)P.r[ii] * (double)P.ug[ii] * (double)P.ug[ii];
        if (P.ug && !of_c && t == 0 && on) {
            double wsum = 0.0;
            for_shared_steps(P.Tn, P.p, i / m, i / m, [&](double wi, double) { wsum += wi; });
            s[u] -= wsum * (double)P.r[i % m] * (double)P.ug[i % m];
        }
        part[16 * t + c] = on ? s[u] : 0.0;
    }
    __syncthreads();
    for (int o = PARTS / 2; o > 0; o >>= 1) {
        for (int e = tid; e < 16 * o; e += FORM_THREADS) part[e] += part[e + 16 * o];
        __syncthreads();
    }
    if (tid < 16) {
        if (of_c) {
            if (tid == 0) *cout = (T)part[0];
        } else if (i < pm) {
            qout[i] = (T)part[c];
        }
    }
}

// Adam refinement of k parents on the quadratic J(z) = z^T P z + 2 q^T z + c
// of a linear problem without the state box: its gradient 2 (P z + q) is
// the rollout cost's gradient exactly (the value the adjoint builds step by
// step), so an Adam step is one product with the symmetric P.  The Adam of
// the adjoint kernel: moments from zero, bias correction, a clamp to the
// knot bounds after every update, and the result kept only if its cost (by
// the same quadratic) is below the entry cost.  The parents are read from
// the population (parameter j of parent b at knots[j ld + idx[b]]) and
// written, refined or not, to Z: [pm][k]; cost_io [k] takes the refined
// costs.  One workgroup per parent, up to QP_MAX_PM parameters.  When P fits
// in the workgroup's LDS (dynamic size pm^2 elements) it is staged there
// once and every product reads it from LDS; otherwise from global memory.
// LS: rows per lane of the product (pm <= 64 LS), a compile-time count so
// the slot loops carry no runtime guards.
constexpr int REF_THREADS = 256, REF_WAVES = REF_THREADS / 64;
constexpr size_t REF_LDS_MAX = 96 * 1024;  // bytes of P staged in LDS at most
template <typename T, int LS>
__global__ __launch_bounds__(REF_THREADS) void qp_refine_kernel(
    int pm, int m, int k, const T *__restrict__ Pg, const T *__restrict__ qv,
    const T *__restrict__ cp, const T *__restrict__ umin, const T *__restrict__ umax, int steps,
    T lr, const T *__restrict__ knots, int64_t ld, const int64_t *__restrict__ idx,
    T *__restrict__ Z, T *__restrict__ cost_io, int p_in_lds) {
    constexpr int REF_SLOTS = (64 * LS + REF_THREADS - 1) / REF_THREADS;
    constexpr int NP = 64 * LS;  // parameters at most
    extern __shared__ __align__(16) unsigned char ref_smem[];
    // the knots in two buffers: an Adam step writes the other one, so one
    // barrier separates it from the next product's reads
    __shared__ T zbuf[2][NP];
    int cur = 0;
    __shared__ double part[REF_WAVES][NP];
    __shared__ double red[REF_WAVES];
    const int tid = threadIdx.x, b = blockIdx.x, lane = tid & 63, wv = tid >> 6;
    T *Pl = (T *)ref_smem;
    const int64_t src = idx[b];
    for (int i = tid; i < pm; i += REF_THREADS) zbuf[0][i] = knots[(int64_t)i * ld + src];
    if (p_in_lds) {
        // P is copied as a flat array: 16-byte pieces, sixteen loads in
        // flight per thread, then their stores (a 140 x 140 FP32 form takes
        // two such rounds per thread); the scalar tail, and every element
        // when P is not 16-byte aligned, one at a time
        typedef T v16 __attribute__((ext_vector_type(16 / sizeof(T))));
        constexpr int W = 16 / sizeof(T);
        const int tot = pm * pm;
        const int nv = (reinterpret_cast<uintptr_t>(Pg) & 15) == 0 ? tot / W : 0;
        const v16 *Pv = reinterpret_cast<const v16 *>(Pg);
        v16 *Lv = reinterpret_cast<v16 *>(Pl);
        for (int e0 = tid; e0 < nv; e0 += 16 * REF_THREADS) {
            v16 t16[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int e = e0 + u * REF_THREADS;
                if (e < nv) t16[u] = Pv[e];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int e = e0 + u * REF_THREADS;
                if (e < nv) Lv[e] = t16[u];
            }
        }
        for (int e = nv * W + tid; e < tot; e += REF_THREADS) Pl[e] = Pg[e];
    }
    // this thread's parameters: linear term and bounds in registers
    T qr[REF_SLOTS], lo[REF_SLOTS], hi[REF_SLOTS];
#pragma unroll
    for (int sl = 0; sl < REF_SLOTS; ++sl) {
        const int i = tid + REF_THREADS * sl;
        qr[sl] = i < pm ? qv[i] : (T)0;
        lo[sl] = i < pm ? umin[i % m] : (T)0;
        hi[sl] = i < pm ? umax[i % m] : (T)0;
    }
    const double c0 = (double)*cp;
    __syncthreads();
    // y = P z: wavefront w sums the columns j of its quarter of 0..pm-1
    // for every row i = lane + 64 s (P symmetric: column j read as row j,
    // contiguous over the lanes), the quarters added in LDS; then, when
    // asked for (the first and the last product: the Adam steps in between
    // need only the gradient), J = sum_i z_i (y_i + 2 q_i) + c over the
    // workgroup.  Each thread returns y for its parameters
    // i = tid + REF_THREADS s.
    double y[REF_SLOTS];
    const int jb = pm * wv / REF_WAVES, je = pm * (wv + 1) / REF_WAVES;
    auto product = [&](bool want_J) {
        // partial sums in the problem's precision, eight columns per pass
        // so that their loads are in flight together
        T acc[LS];
#pragma unroll
        for (int sl = 0; sl < LS; ++sl) acc[sl] = 0;
        // P from LDS or from global memory, each loop on its own pointer so
        // that the LDS one compiles to LDS reads
        auto columns = [&](const T *Pp) {
#pragma unroll 8
            for (int j = jb; j < je; ++j) {
                const T zj = zbuf[cur][j];
                const T *row = Pp + (int64_t)j * pm;
#pragma unroll
                for (int sl = 0; sl < LS; ++sl) {
                    const int i = lane + 64 * sl;
                    acc[sl] += (i < pm ? row[i] : (T)0) * zj;
                }
            }
        };
        if (p_in_lds)
            columns(Pl);
        else
            columns(Pg);
#pragma unroll
        for (int sl = 0; sl < LS; ++sl) {
            const int i = lane + 64 * sl;
            if (i < pm) part[wv][i] = (double)acc[sl];
        }
        __syncthreads();
        double pj = 0.0;
#pragma unroll
        for (int sl = 0; sl < REF_SLOTS; ++sl) {
            const int i = tid + REF_THREADS * sl;
            double a = 0.0;
            if (i < pm) {
#pragma unroll
                for (int w2 = 0; w2 < REF_WAVES; ++w2) a += part[w2][i];
                pj += (double)zbuf[cur][i] * (a + 2.0 * (double)qr[sl]);
            }
            y[sl] = a;
        }
        if (!want_J) return 0.0;  // uniform over the workgroup
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) pj += __shfl_xor(pj, o, 64);
        if (lane == 0) red[wv] = pj;
        __syncthreads();
        double J = c0;
#pragma unroll
        for (int w2 = 0; w2 < REF_WAVES; ++w2) J += red[w2];
        return J;
    };
    const T b1 = (T)0.9, b2 = (T)0.999, eps = (T)1e-8;
    T b1t = 1, b2t = 1;
    T m1[REF_SLOTS], m2[REF_SLOTS];
#pragma unroll
    for (int sl = 0; sl < REF_SLOTS; ++sl) m1[sl] = m2[sl] = 0;
    double J0 = 0.0;
    for (int t = 1; t <= steps; ++t) {
        const double Jt = product(t == 1);
        if (t == 1) J0 = Jt;
        b1t *= b1;
        b2t *= b2;
        T U[REF_SLOTS];
#pragma unroll
        for (int sl = 0; sl < REF_SLOTS; ++sl) {
            const int i = tid + REF_THREADS * sl;
            if (i < pm) {
                const T g = (T)(2.0 * (y[sl] + (double)qr[sl]));
                m1[sl] = b1 * m1[sl] + ((T)1 - b1) * g;
                m2[sl] = b2 * m2[sl] + ((T)1 - b2) * g * g;
                const T mh = m1[sl] / ((T)1 - b1t), vh = m2[sl] / ((T)1 - b2t);
                T u = zbuf[cur][i] - lr * mh / (sqrt(vh) + eps);
                u = u < lo[sl] ? lo[sl] : u;
                u = u > hi[sl] ? hi[sl] : u;
                U[sl] = u;
            }
        }
        // every read of the current buffer lies before this step's product
        // barrier or is this thread's own; the next product reads the other
#pragma unroll
        for (int sl = 0; sl < REF_SLOTS; ++sl) {
            const int i = tid + REF_THREADS * sl;
            if (i < pm) zbuf[cur ^ 1][i] = U[sl];
        }
        cur ^= 1;
        __syncthreads();
    }
    const double Jn = product(true);
    const bool keep = steps > 0 && Jn < J0;  // uniform over the workgroup
    for (int i = tid; i < pm; i += REF_THREADS)
        Z[(int64_t)i * k + b] = keep ? zbuf[cur][i] : knots[(int64_t)i * ld + src];
    if (keep && tid == 0) cost_io[b] = (T)Jn;
}

// sum over the workgroup (every thread gets it)
__device__ inline double block_sum(double x, double *red) {
    red[threadIdx.x] = x;
    __syncthreads();
    for (int o = QP_THREADS / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const double t = red[0];
    __syncthreads();
    return t;
}

// max over the workgroup (every thread gets it)
__device__ inline double block_max(double x, double *red) {
    red[threadIdx.x] = x;
    __syncthreads();
    for (int o = QP_THREADS / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + o]);
        __syncthreads();
    }
    const double t = red[0];
    __syncthreads();
    return t;
}

// Box QP min f(z) = z^T P z + 2 q^T z, lo <= z <= hi, by Bertsekas' projected
// Newton method (SIAM J. Control Optim. 20, 1982): with g = 2 (P z + q) and
// w = |z - clip(z - g)|_inf, the variables within min(eps, w) of a bound
// whose gradient points out of the box are held on a scaled gradient step,
// the rest take the Newton step of the reduced quadratic (a Cholesky solve
// of P on the free variables), and the step is cut back along the
// projection arc until the Armijo condition f(z) - f(z') >= sigma g^T (z -
// z') holds.  Globally convergent for a positive definite P; once the active
// set is the optimal one the full Newton step lands on the minimizer.
template <typename T>
__global__ __launch_bounds__(QP_THREADS) void qp_box_kernel(
    int pm, int m, const T *__restrict__ umin, const T *__restrict__ umax,
    const T *__restrict__ Pm, const T *__restrict__ qv, const T *__restrict__ cp, int max_iter,
    double *__restrict__ H, T *__restrict__ zout, T *__restrict__ cost, int *__restrict__ info) {
    __shared__ double z[QP_MAX_PM], d[QP_MAX_PM], y[QP_MAX_PM], red[QP_THREADS];
    __shared__ int act[QP_MAX_PM], idx[QP_MAX_PM], s_nfree;
    const int i = threadIdx.x;
    const bool mine = i < pm;
    const double lo = mine ? (double)umin[i % m] : 0.0, hi = mine ? (double)umax[i % m] : 0.0;
    const double qi = mine ? (double)qv[i] : 0.0;
    const double pii = mine ? (double)Pm[(int64_t)i * pm + i] : 1.0;
    auto clip = [&](double v) { return v < lo ? lo : (v > hi ? hi : v); };
    // (P v)_i for v in LDS
    auto pdot = [&](const double *v) {
        double s = 0.0;
        if (mine)
            for (int j = 0; j < pm; ++j) s += (double)Pm[(int64_t)i * pm + j] * v[j];
        return s;
    };
    if (mine) z[i] = clip(0.0);
    __syncthreads();
    double pz = pdot(z);
    double f = block_sum(mine ? z[i] * (pz + 2.0 * qi) : 0.0, red);
    int it = 0, converged = 0;
    const double eps0 = 1e-3;
    for (; it < max_iter; ++it) {
        const double g = mine ? 2.0 * (pz + qi) : 0.0;
        const double w = block_max(mine ? fabs(z[i] - clip(z[i] - g)) : 0.0, red);
        const double gs = block_max(mine ? fabs(g) : 0.0, red);
        if (w <= 1e-14 * (1.0 + gs)) {
            converged = 1;
            break;
        }
        const double eps = w < eps0 ? w : eps0;
        int a = 0;
        if (mine) a = (z[i] <= lo + eps && g > 0.0) || (z[i] >= hi - eps && g < 0.0);
        if (mine) act[i] = a;
        __syncthreads();
        if (i == 0) {
            int c = 0;
            for (int t = 0; t < pm; ++t)
                if (!act[t]) idx[c++] = t;
            s_nfree = c;
        }
        __syncthreads();
        const int nf = s_nfree;
        // Newton step on the free variables: P_FF d_F = -(P z + q)_F
        for (int e = i; e < nf * nf; e += QP_THREADS) {
            const int r = e / nf, c = e % nf;
            H[e] = (double)Pm[(int64_t)idx[r] * pm + idx[c]];
        }
        if (mine && !a) d[i] = -(pz + qi);  // gathered below
        if (mine && a) d[i] = -g / (2.0 * pii);
        __syncthreads();
        if (i < nf) y[i] = d[idx[i]];
        __syncthreads();
        for (int k = 0; k < nf; ++k) {
            if (i == 0) H[k * nf + k] = sqrt(H[k * nf + k]);
            __syncthreads();
            const double dk = H[k * nf + k];
            for (int r = k + 1 + i; r < nf; r += QP_THREADS) H[r * nf + k] /= dk;
            __syncthreads();
            const int wdt = nf - k - 1;
            for (int e = i; e < wdt * wdt; e += QP_THREADS) {
                const int r = k + 1 + e / wdt, c = k + 1 + e % wdt;
                if (c <= r) H[r * nf + c] -= H[r * nf + k] * H[c * nf + k];
            }
            __syncthreads();
        }
        for (int k = 0; k < nf; ++k) {
            if (i == 0) y[k] /= H[k * nf + k];
            __syncthreads();
            for (int r = k + 1 + i; r < nf; r += QP_THREADS) y[r] -= H[r * nf + k] * y[k];
            __syncthreads();
        }
        for (int k = nf - 1; k >= 0; --k) {
            if (i == 0) y[k] /= H[k * nf + k];
            __syncthreads();
            for (int r = i; r < k; r += QP_THREADS) y[r] -= H[k * nf + r] * y[k];
            __syncthreads();
        }
        if (i < nf) d[idx[i]] = y[i];
        __syncthreads();
        // Armijo search along the projection arc
        const double z_old = mine ? z[i] : 0.0;
        double alpha = 1.0, pz_new = pz, f_new = f;
        bool moved = false;
        for (int ls = 0; ls < 60; ++ls) {
            const double zt = mine ? clip(z_old + alpha * d[i]) : 0.0;
            __syncthreads();
            if (mine) y[i] = zt;
            __syncthreads();
            pz_new = pdot(y);
            f_new = block_sum(mine ? zt * (pz_new + 2.0 * qi) : 0.0, red);
            const double dec = block_sum(mine ? g * (z_old - zt) : 0.0, red);
            if (f - f_new >= 1e-4 * dec) {
                moved = true;
                break;
            }
            alpha *= 0.5;
        }
        if (!moved) {  // no decrease left at rounding level
            converged = 1;
            break;
        }
        // a step below rounding of z: nothing left to gain
        const double step = block_max(mine ? fabs(y[i] - z_old) : 0.0, red);
        const double zmax = block_max(mine ? fabs(z_old) : 0.0, red);
        if (mine) z[i] = y[i];
        pz = pz_new;
        f = f_new;
        __syncthreads();
        if (step <= 1e-15 * (1.0 + zmax)) {
            converged = 1;
            ++it;
            break;
        }
    }
    if (mine) zout[i] = (T)z[i];
    if (i == 0) {
        *cost = (T)(f + (double)*cp);
        info[0] = it;
        info[1] = converged;
    }
}

// The same method with the factor in LDS, up to BOX_MAX_PM parameters: the
// same operations on every element in the same order, so the same iterates.
// What bounds it is the chain of a Cholesky column (pivot square root,
// reciprocal, scaling, the next pivot's update).  The lower triangle sits in
// block rows of 16 rows (block row I: 16 (I + 1) columns, two of padding, so
// that a column read by 16 rows falls in different banks); the right-hand
// side is one more row of it, so the forward substitution is part of the
// factorization; a last block is filled up with rows of the identity, which
// couple to nothing.  A panel of 16 columns is eliminated in registers, a row
// per lane: every wavefront carries the panel's 16 diagonal rows and 48
// others, so the panel needs no barrier and pivots move by lane reads; the
// trailing tiles are then updated on the FP64 matrix cores, those of the next
// panel's columns first, the others by the idle wavefronts while that panel
// runs.  P is transposed once into the workspace, so that P z, a serial sum
// per row, reads contiguous lanes (from the matrix cores with P read or
// staged in their operand layout it took longer: 64 cycles for four terms).
// 140 parameters, 4 Newton steps: 1124 us with the factor in global memory
// and three barriers per column, 141 us here.
constexpr int BOX_MAX_PM = 160;  // with the right-hand side's 11 block rows: 138 KB of LDS
constexpr int BOX_WAVES = 8, BOX_THREADS = 64 * BOX_WAVES;

__host__ __device__ constexpr int box_row(int r) {
    const int I = r >> 4;
    return 16 * (8 * I * (I + 1) + 2 * I) + (r & 15) * (16 * (I + 1) + 2);
}
// block rows of pm rows and one for the right-hand side; at first the columns
// of P that are transposed at a time
constexpr int BOX_STAGE = 64;
__host__ __device__ inline size_t box_lds_doubles(int pm) {
    const size_t h = box_row(16 * ((pm + 15) / 16 + 1));
    const size_t st = (size_t)(pm < BOX_STAGE ? pm : BOX_STAGE) * (pm + 1);
    return h > st ? h : st;
}

// A pivot's square root d, and r within 2^-44 of 1 / d, come from one hardware
// estimate of the inverse root (about 23 bits): a coupled Newton step for
// root and half inverse, then one correction of the root by its exact fused
// residual; a / d is a r corrected once by the quotient's exact residual.  In
// the plain range both agree with sqrt and the division on every one of 2e9
// random and near-square values, in a third of their dependent instructions.
struct Pivot {
    double d, r;
};
__device__ __forceinline__ double quotient(double a, const Pivot &p) {
    const double q = a * p.r;
    return fma(fma(-p.d, q, a), p.r, q);
}
// pivots whose root and quotients stay clear of under- and overflow
__device__ __forceinline__ bool plain_range(double d) { return d > 1e-100 && d < 1e100; }

// Sixteen columns eliminated in the registers l of the panel's rows (lane k <
// 16: the diagonal rows).  Returns whether every pivot was in the plain range.
// The chain from one column to the next (pivot, root, quotient, the next
// column's update: about 130 cycles) leaves issue slots free, which the
// other columns' updates fill: two of them, lane reads and multiply-adds, are
// fixed between the chain's stages.
__device__ __forceinline__ bool eliminate_panel(double *l, bool first, double *dg, double *rv) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // its comparisons stay here: hoisted masks spill
    bool plain = true;
    Pivot own = {0.0, 0.0};  // lane k keeps pivot k
    double q = 0.0;          // column k - 1, which the columns past k have not seen yet
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        auto update = [&](int c0) {  // columns c0, c0 + 1 by column k - 1
#pragma unroll
            for (int c = c0; c < c0 + 2; ++c)
                if (k > 0 && c < 16) l[c] = fma(-q, lane_bcast<double>(q, c), l[c]);
            __builtin_amdgcn_sched_barrier(0);
        };
        const double a = lane_bcast<double>(l[k], k);
        const double y = __builtin_amdgcn_rsq(a);
        update(k + 1);
        const double g = a * y, h = 0.5 * y;
        update(k + 3);
        const double e = fma(-h, g, 0.5);
        update(k + 5);
        const double g1 = fma(g, e, g), h1 = fma(h, e, h);
        update(k + 7);
        const double res = fma(-g1, g1, a);
        Pivot p;
        p.r = h1 + h1;
        const double q0 = l[k] * p.r;
        update(k + 9);
        p.d = fma(res, h1, g1);
        update(k + 11);
        const double rem = fma(-p.d, q0, l[k]);
        update(k + 13);
        // (the pivot's own row right of the pivot is never read again)
        q = fma(rem, p.r, q0);
        l[k] = lane == k ? p.d : q;
        own.d = lane == k ? p.d : own.d;
        own.r = lane == k ? p.r : own.r;
        plain = plain && plain_range(p.d);
        if (k < 15) l[k + 1] = fma(-q, lane_bcast<double>(q, k + 1), l[k + 1]);
    }
    if (first && lane < 16) {
        dg[lane] = own.d;
        rv[lane] = own.r;
    }
    return plain;
}

template <typename T>
__global__ __launch_bounds__(BOX_THREADS) void qp_box_small_kernel(
    int pm, int m, const T *__restrict__ umin, const T *__restrict__ umax,
    const T *__restrict__ Pm, const T *__restrict__ qv, const T *__restrict__ cp, int max_iter,
    double *__restrict__ PT, T *__restrict__ zout, T *__restrict__ cost, int *__restrict__ info) {
    extern __shared__ __align__(16) double H[];
    __shared__ double z[192], d[192], y[192], dg[192], rv[192], pv[192];
    __shared__ double red[2][2][192];
    __shared__ int idx[192], cnt[4], s_plain;
    const int i = threadIdx.x, lane = i & 63;
    const int wave = __builtin_amdgcn_readfirstlane(i >> 6);
    const bool mine = i < pm;
    const double lo = mine ? (double)umin[i % m] : 0.0, hi = mine ? (double)umax[i % m] : 0.0;
    const double qi = mine ? (double)qv[i] : 0.0;
    const double pii = mine ? (double)Pm[(int64_t)i * pm + i] : 1.0;
    auto clip = [&](double v) { return v < lo ? lo : (v > hi ? hi : v); };
    const int cl = lane & 15, gr = lane >> 4;
    // PT[j][i] = P[i][j], BOX_STAGE columns at a time through LDS, eight rows
    // of a wavefront in flight
    for (int c0 = 0; c0 < pm; c0 += BOX_STAGE) {
        const int nc = min(pm - c0, BOX_STAGE), c = min(lane, nc - 1);
        for (int r0 = wave; r0 < pm; r0 += 8 * BOX_WAVES) {
            T t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                t[u] = Pm[(int64_t)min(r0 + u * BOX_WAVES, pm - 1) * pm + c0 + c];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int r = r0 + u * BOX_WAVES;
                if (lane < nc && r < pm) H[lane * (pm + 1) + r] = (double)t[u];
            }
        }
        __syncthreads();
        for (int k = wave; k < nc; k += BOX_WAVES)
            for (int r = lane; r < pm; r += 64)
                PT[(int64_t)(c0 + k) * pm + r] = H[k * (pm + 1) + r];
        __syncthreads();
    }
    // (P v)_i for v in LDS.  Twenty loads in flight, the rest one more batch of
    // them with clamped rows: a thread waits for memory once per batch, and a
    // longer batch does more beyond the last row.  16, 20, 24, 32 loads, us per
    // solve: 49 parameters 39, 40, 39, 42; 100 75, 72, 75, 78; 140 124, 121,
    // 125, 129; 160 121, 120, 124, 124.
    auto pdot = [&](const double *v) {
        double s = 0.0;
        if (mine) {
            const double *col = PT + i;
            int j = 0;
            constexpr int U = 20;
            for (; j + U <= pm; j += U) {
                double t[U];
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] = col[(int64_t)(j + u) * pm];
#pragma unroll
                for (int u = 0; u < U; ++u) s += t[u] * v[j + u];
            }
            if (j < pm) {
                double t[U];
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] = col[(int64_t)min(j + u, pm - 1) * pm];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (j + u < pm) s += t[u] * v[j + u];
            }
        }
        return s;
    };
    // two sums (or maxima) over the threads i < 192 at once, in every thread:
    // wavefronts 0 + 2, then + 1, then lanes in halves (32 and 16 apart from
    // LDS, the rest by row shifts).  Alternating buffers: one barrier each.
    int rb = 0;
    auto reduce = [&](double a, double b, auto &&op, double *ra, double *rbv) {
        if (i < 192) {
            red[rb][0][i] = a;
            red[rb][1][i] = b;
        }
        __syncthreads();
        auto tree = [&](const double *x) {
            const int t = lane & 15;
            double w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                w[u] = op(op(x[t + 16 * u], x[t + 16 * u + 128]), x[t + 16 * u + 64]);
            double s = op(op(w[0], w[2]), op(w[1], w[3]));
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) s = op(s, row_shift_down<double>(s, o));
            return lane_bcast<double>(s, 0);
        };
        *ra = tree(red[rb][0]);
        *rbv = tree(red[rb][1]);
        rb ^= 1;
    };
    auto add = [](double a, double b) { return a + b; };
    auto max2 = [](double a, double b) { return fmax(a, b); };
    if (i < 192) {
        z[i] = mine ? clip(0.0) : 0.0;
        y[i] = 0.0;
    }
    __syncthreads();
    double pz = pdot(z);
    double f, unused;
    reduce(mine ? z[i] * (pz + 2.0 * qi) : 0.0, 0.0, add, &f, &unused);
    int it = 0, converged = 0;
    const double eps0 = 1e-3;
    for (; it < max_iter; ++it) {
        const double g = mine ? 2.0 * (pz + qi) : 0.0;
        double w, gs;
        reduce(mine ? fabs(z[i] - clip(z[i] - g)) : 0.0, mine ? fabs(g) : 0.0, max2, &w, &gs);
        if (w <= 1e-14 * (1.0 + gs)) {
            converged = 1;
            break;
        }
        const double eps = w < eps0 ? w : eps0;
        int a = 0;
        if (mine) a = (z[i] <= lo + eps && g > 0.0) || (z[i] >= hi - eps && g < 0.0);
        // the free variables in ascending order
        const unsigned long long fm = __ballot(mine && !a);
        if (lane == 0 && wave < 3) cnt[wave] = __popcll(fm);
        __syncthreads();
        const int nf = cnt[0] + cnt[1] + cnt[2];
        // position of variable i among the free ones
        const int at = (wave > 0 ? cnt[0] : 0) + (wave > 1 ? cnt[1] : 0) +
                       __popcll(fm & ((1ull << lane) - 1));
        if (mine && a) d[i] = -g / (2.0 * pii);
        if (mine && !a) idx[at] = i;
        if (i == 0) s_plain = 1;
        __syncthreads();
        const int np = (nf + 15) / 16, nr = 16 * np;  // panels; the right-hand side's row
        // one trailing tile: (I, K) minus L_IJ L_KJ^T
        auto tile = [&](int I, int K, int J) {
            const int sI = 16 * (I + 1) + 2, sK = 16 * (K + 1) + 2;  // row strides
            const double *A = H + box_row(16 * I) + cl * sI + 16 * J + gr;
            const double *B = H + box_row(16 * K) + cl * sK + 16 * J + gr;
            double *C = H + box_row(16 * I) + gr * sI + 16 * K + cl;
            v4d acc;
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] = C[4 * v * sI];
#pragma unroll
            for (int k = 0; k < 16; k += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-A[k], B[k], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) C[4 * v * sI] = acc[v];
        };
        auto gather = [&]() {
            // Newton step on the free variables: P_FF d_F = -(P z + q)_F, the
            // right-hand side as the last row; four rows of a wavefront in flight
            if (mine && !a) H[box_row(nr) + at] = -(pz + qi);
            if (i >= nf && i < nr) {  // fill-up rows
                H[box_row(nr) + i] = 0.0;
                for (int c = 0; c < i; ++c) H[box_row(i) + c] = 0.0;
                H[box_row(i) + i] = 1.0;
            }
            for (int r0 = wave; r0 < nf; r0 += 4 * BOX_WAVES) {
                T t[4][3];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int r = r0 + u * BOX_WAVES < nf ? r0 + u * BOX_WAVES : r0;
                    const T *row = Pm + (int64_t)idx[r] * pm;
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if (64 * q <= r) t[u][q] = row[idx[lane + 64 * q < r ? lane + 64 * q : r]];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int r = r0 + u * BOX_WAVES;
                    if (r >= nf) continue;
                    double *to = H + box_row(r);
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if (lane + 64 * q <= r) to[lane + 64 * q] = (double)t[u][q];
                }
            }
            __syncthreads();
        };
        gather();
        for (int J = 0; J < np; ++J) {
            const int c0 = 16 * J, below = nr + 1 - (c0 + 16);  // rows under the diagonal block
            const int nw = (below + 47) / 48;
            const int r = lane < 16 ? c0 + lane : c0 + 48 * wave + lane;
            const bool live = lane < 16 ? wave == 0 : r <= nr;
            double *row = H + box_row(lane < 16 || r <= nr ? r : nr) + c0;
            double l[16];
            if (wave < nw) {
#pragma unroll
                for (int k = 0; k < 16; ++k) l[k] = row[k];
            }
            __syncthreads();  // every wavefront reads the diagonal rows, the first stores them
            if (wave < nw) {
                const bool plain = eliminate_panel(l, wave == 0, dg + c0, rv + c0);
                if (wave == 0 && lane == 0 && !plain) s_plain = 0;
                if (live) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) row[k] = l[k];
                }
            } else if (J > 0) {
                // meanwhile the other wavefronts finish panel J - 1's update
                // right of this panel (the panel's own column came first)
                int t = 0;
                for (int K = J + 1; K < np; ++K)
                    for (int I = K; I <= np; ++I, ++t)
                        if (t % (BOX_WAVES - nw) == wave - nw) tile(I, K, J - 1);
            }
            __syncthreads();
            if (J + 1 < np)  // the next panel's column
                for (int I = J + 1 + wave; I <= np; I += BOX_WAVES) tile(I, J + 1, J);
            __syncthreads();
        }
        if (s_plain) {  // uniform: written before the last barrier
            // L^T d = y, thread i < nr with entry i, 16 unknowns at a time: the
            // wavefront that holds them solves the diagonal block by lane
            // reads and publishes them, then every entry below them in index
            // takes the 16 updates, in descending order as the plain
            // substitution does (what they read of L is loaded beforehand)
            double yv = i < nr ? H[box_row(nr) + i] : 0.0;
            for (int J = np - 1; J >= 0; --J) {
                const int c0 = 16 * J, l0 = c0 & 63;
                double *qs = red[J & 1][0];
                double lk[16];
                if (wave < 3) {
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        lk[k] = H[box_row(c0 + k) + (i < c0 + 15 ? i : c0 + 15)];
                }
                if (wave == J / 4) {
                    int bc = lane - l0;  // column in the block, lanes l0 .. l0 + 15
                    asm volatile("" : "+v"(bc));  // as in eliminate_panel
                    const Pivot p = {dg[i], rv[i]};
                    double y = yv;
#pragma unroll
                    for (int k = 15; k >= 0; --k) {
                        const double q = quotient(y, p);
                        const double qk = lane_bcast<double>(q, l0 + k);
                        y = fma(-lk[k], qk, y);  // of no use from entry k on
                        yv = bc == k ? q : yv;
                    }
                    if (bc >= 0 && bc < 16) qs[bc] = yv;
                }
                __syncthreads();
                if (i < c0) {
#pragma unroll
                    for (int k = 15; k >= 0; --k) yv = fma(-lk[k], qs[k], yv);
                }
            }
            if (i < 192) pv[i] = yv;
        } else {
            // pivots near under- or overflow (or not positive): the plain
            // column algorithm with the library's square root and division
            __syncthreads();
            gather();
            for (int k = 0; k < nf; ++k) {
                if (i == 0) H[box_row(k) + k] = sqrt(H[box_row(k) + k]);
                __syncthreads();
                const double dk = H[box_row(k) + k];
                for (int r = k + 1 + i; r <= nr; r += BOX_THREADS) H[box_row(r) + k] /= dk;
                __syncthreads();
                for (int r = k + 1 + wave; r <= nr; r += BOX_WAVES)
                    for (int c = k + 1 + lane; c <= r && c < nf; c += 64)
                        H[box_row(r) + c] -= H[box_row(r) + k] * H[box_row(c) + k];
                __syncthreads();
            }
            double *ys = H + box_row(nr);
            for (int k = nf - 1; k >= 0; --k) {
                if (i == 0) ys[k] /= H[box_row(k) + k];
                __syncthreads();
                if (i < k) ys[i] -= H[box_row(k) + i] * ys[k];
                __syncthreads();
            }
            if (i < nf) pv[i] = ys[i];
        }
        __syncthreads();
        if (mine && !a) d[i] = pv[at];
        // Armijo search along the projection arc
        const double z_old = mine ? z[i] : 0.0;
        double alpha = 1.0, pz_new = pz, f_new = f;
        bool moved = false;
        for (int ls = 0; ls < 60; ++ls) {
            const double zt = mine ? clip(z_old + alpha * d[i]) : 0.0;
            if (mine) y[i] = zt;  // read again only after the reduction's barrier below
            __syncthreads();
            pz_new = pdot(y);
            double dec;
            reduce(mine ? zt * (pz_new + 2.0 * qi) : 0.0, mine ? g * (z_old - zt) : 0.0, add,
                   &f_new, &dec);
            if (f - f_new >= 1e-4 * dec) {
                moved = true;
                break;
            }
            alpha *= 0.5;
        }
        if (!moved) {  // no decrease left at rounding level
            converged = 1;
            break;
        }
        // a step below rounding of z: nothing left to gain
        double step, zmax;
        reduce(mine ? fabs(y[i] - z_old) : 0.0, mine ? fabs(z_old) : 0.0, max2, &step, &zmax);
        if (mine) z[i] = y[i];
        pz = pz_new;
        f = f_new;
        if (step <= 1e-15 * (1.0 + zmax)) {
            converged = 1;
            ++it;
            break;
        }
    }
    if (mine) zout[i] = (T)z[i];
    if (i == 0) {
        *cost = (T)(f + (double)*cp);
        info[0] = it;
        info[1] = converged;
    }
}

}  // namespace

// workspace of the form, in doubles: S [T n][pm], v [T n]; the box solver
// adds P transposed (above BOX_MAX_PM parameters the factor) [pm][pm]
static size_t form_doubles(int n, int T, int pm) {
    const size_t S = (size_t)T * n * pm, v = (size_t)T * n;
    return (S + 31) / 32 * 32 + (v + 31) / 32 * 32;
}

size_t qp_workspace_bytes(int n, int T, int pm) {
    return (form_doubles(n, T, pm) + (size_t)pm * pm) * sizeof(double);
}

template <typename T>
hipError_t launch_qp_form(const ProbView<T> &P, const T *x0, void *ws, T *Pout, T *qout, T *cout,
                          hipStream_t s) {
    const int pm = P.p * P.m, n = P.n;
    double *S = (double *)ws;
    double *v = S + ((size_t)P.Tn * n * pm + 31) / 32 * 32;
    // register row lengths; one wavefront up to 64 states (its barriers cost
    // nothing), two above
    if (n <= 16)
        hipLaunchKernelGGL((qp_traj_kernel<T, 16, 64>), dim3(pm + 1), dim3(64), 0, s, P, x0, S, v);
    else if (n <= 32)
        hipLaunchKernelGGL((qp_traj_kernel<T, 32, 64>), dim3(pm + 1), dim3(64), 0, s, P, x0, S, v);
    else if (n <= 64)
        hipLaunchKernelGGL((qp_traj_kernel<T, 64, 64>), dim3(pm + 1), dim3(64), 0, s, P, x0, S, v);
    else
        hipLaunchKernelGGL((qp_traj_kernel<T, 80, 128>), dim3(pm + 1), dim3(128), 0, s, P, x0, S,
                           v);
    const int tiles = (pm + 15) / 16;
    hipLaunchKernelGGL(qp_form_kernel<T>, dim3((unsigned)(tiles * (tiles + 1) + 1)),
                       dim3(FORM_THREADS), 0, s, P, S, v, tiles, Pout, qout, cout);
    return hipGetLastError();
}

size_t qp_form_bytes(int n, int T, int pm) { return form_doubles(n, T, pm) * sizeof(double); }

template <typename T>
hipError_t launch_qp_refine(const ProbView<T> &P, const T *Pm, const T *q, const T *c,
                            const T *knots, int64_t ld, const int64_t *idx, T *Z, int k,
                            int steps, T lr, T *cost_io, hipStream_t s) {
    const int pm = P.p * P.m;
    const size_t bytes = (size_t)pm * pm * sizeof(T);
    const int in_lds = bytes <= REF_LDS_MAX ? 1 : 0;
    const size_t dyn = in_lds ? bytes : 0;
    auto go = [&](auto kernel) {
        if (dyn > 65536) {
            const hipError_t e = hipFuncSetAttribute((const void *)kernel,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)dyn);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3(k), dim3(REF_THREADS), dyn, s, pm, P.m, k, Pm, q, c,
                           P.umin, P.umax, steps, lr, knots, ld, idx, Z, cost_io, in_lds);
        return hipGetLastError();
    };
    if (pm <= 64) return go(qp_refine_kernel<T, 1>);
    if (pm <= 128) return go(qp_refine_kernel<T, 2>);
    if (pm <= 256) return go(qp_refine_kernel<T, 4>);
    if (pm <= 512) return go(qp_refine_kernel<T, 8>);
    return go(qp_refine_kernel<T, 16>);
}
template hipError_t launch_qp_refine<float>(const ProbView<float> &, const float *, const float *,
                                            const float *, const float *, int64_t,
                                            const int64_t *, float *, int, int, float, float *,
                                            hipStream_t);
template hipError_t launch_qp_refine<double>(const ProbView<double> &, const double *,
                                             const double *, const double *, const double *,
                                             int64_t, const int64_t *, double *, int, int, double,
                                             double *, hipStream_t);

template <typename T>
hipError_t launch_qp_solve(const ProbView<T> &P, const T *Pm, const T *q, const T *c, void *ws,
                           int max_iter, T *z, T *cost, int *info, hipStream_t s) {
    const int pm = P.p * P.m, n = P.n;
    double *H = (double *)ws + form_doubles(n, P.Tn, pm);
    // the factor and its right-hand side fit in LDS up to BOX_MAX_PM
    if (pm <= BOX_MAX_PM) {
        const size_t bytes = box_lds_doubles(pm) * sizeof(double);
        if (bytes > 49152) {
            const hipError_t e = hipFuncSetAttribute((const void *)qp_box_small_kernel<T>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)bytes);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(qp_box_small_kernel<T>, dim3(1), dim3(BOX_THREADS), bytes, s, pm, P.m,
                           P.umin, P.umax, Pm, q, c, max_iter, H, z, cost, info);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(qp_box_kernel<T>, dim3(1), dim3(QP_THREADS), 0, s, pm, P.m, P.umin, P.umax,
                       Pm, q, c, max_iter, H, z, cost, info);
    return hipGetLastError();
}

template hipError_t launch_qp_form<float>(const ProbView<float> &, const float *, void *, float *,
                                          float *, float *, hipStream_t);
template hipError_t launch_qp_form<double>(const ProbView<double> &, const double *, void *,
                                           double *, double *, double *, hipStream_t);
template hipError_t launch_qp_solve<float>(const ProbView<float> &, const float *, const float *,
                                           const float *, void *, int, float *, float *, int *,
                                           hipStream_t);
template hipError_t launch_qp_solve<double>(const ProbView<double> &, const double *,
                                            const double *, const double *, void *, int, double *,
                                            double *, int *, hipStream_t);

}  // namespace empc

using namespace empc;

empc_status empc_validate_problem_internal(const empc_problem *P);
empc_status empc_fail_internal(empc_status s, const char *msg);

namespace {

empc_status check_qp_problem(const empc_problem *P) {
    empc_status st = empc_validate_problem_internal(P);
    if (st) return st;
    if (P->model != EMPC_LINEAR)
        return empc_fail_internal(EMPC_EUNSUPPORTED, "the convex form needs a linear model");
    if (P->qb) return empc_fail_internal(EMPC_EUNSUPPORTED, "the state box penalty is not quadratic");
    if (P->Q || P->R || P->Qf)
        return empc_fail_internal(EMPC_EUNSUPPORTED, "the convex form takes diagonal weights");
    if (P->p * P->m > QP_MAX_PM)
        return empc_fail_internal(EMPC_EUNSUPPORTED, "more than 1024 knot parameters");
    return EMPC_OK;
}

empc_status qp_launched(hipError_t e) {
    if (e == hipSuccess) return EMPC_OK;
    return empc_fail_internal(EMPC_EDEVICE, hipGetErrorString(e));
}

}  // namespace

extern "C" {

size_t empc_qp_workspace_bytes(const empc_problem *prob) {
    if (check_qp_problem(prob)) return 0;
    return qp_workspace_bytes(prob->n, prob->T, prob->p * prob->m);
}

empc_status empc_qp_form(const empc_problem *prob, const void *x0, void *workspace,
                         size_t ws_bytes, void *P, void *q, void *c, void *stream) {
    empc_status st = check_qp_problem(prob);
    if (st) return st;
    if (!x0 || !P || !q || !c) return empc_fail_internal(EMPC_EINVAL, "x0, P, q and c are required");
    if (!workspace || ws_bytes < qp_workspace_bytes(prob->n, prob->T, prob->p * prob->m))
        return empc_fail_internal(EMPC_EWORKSPACE, "convex workspace too small");
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return qp_launched(e);
    hipStream_t s = (hipStream_t)stream;
    if (prob->dtype == EMPC_F32)
        e = launch_qp_form<float>(view_of<float>(*prob), (const float *)x0, workspace, (float *)P,
                                  (float *)q, (float *)c, s);
    else
        e = launch_qp_form<double>(view_of<double>(*prob), (const double *)x0, workspace,
                                   (double *)P, (double *)q, (double *)c, s);
    return qp_launched(e);
}

empc_status empc_qp_solve(const empc_problem *prob, const void *P, const void *q, const void *c,
                          void *workspace, size_t ws_bytes, int32_t max_iter, void *z, void *cost,
                          int32_t *info, void *stream) {
    empc_status st = check_qp_problem(prob);
    if (st) return st;
    if (!P || !q || !c || !z || !cost || !info)
        return empc_fail_internal(EMPC_EINVAL, "P, q, c, z, cost and info are required");
    if (max_iter < 1) return empc_fail_internal(EMPC_EINVAL, "max_iter must be >= 1");
    if (!workspace || ws_bytes < qp_workspace_bytes(prob->n, prob->T, prob->p * prob->m))
        return empc_fail_internal(EMPC_EWORKSPACE, "convex workspace too small");
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return qp_launched(e);
    hipStream_t s = (hipStream_t)stream;
    if (prob->dtype == EMPC_F32)
        e = launch_qp_solve<float>(view_of<float>(*prob), (const float *)P, (const float *)q,
                                   (const float *)c, workspace, max_iter, (float *)z,
                                   (float *)cost, (int *)info, s);
    else
        e = launch_qp_solve<double>(view_of<double>(*prob), (const double *)P, (const double *)q,
                                    (const double *)c, workspace, max_iter, (double *)z,
                                    (double *)cost, (int *)info, s);
    return qp_launched(e);
}

}  // extern "C"
