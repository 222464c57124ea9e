// N-link planar robot (gfx950): the robot of the paper's convex-solver and
// EMPC experiments (Sec. IV-F setup, Sec. VI-A), M(q) qdd + C(q, qd) + b qd
// = tau, in a plane perpendicular to gravity, point masses at the link ends.
// EMPC runs on a linear model (eq. 2) relinearized at the current state
// every control tick; these kernels produce that model on the device and
// simulate the robot itself:
//  - nlink_linearize_kernel: the exact Jacobians of f(x, tau) = [qd; qdd] at
//    (x, u), the affine offset, and the zero-order hold over dt
//    (A_d, B_d, w_d from the exponential of [[A, B, w], [0, 0, 0]] dt);
//  - nlink_step_kernel: classical RK4 substeps of the nonlinear dynamics.
//
// Both work in the absolute angles th_a = q_0 + .. + q_a (rates om_a, torque
// on th_a: tau_a - tau_{a+1}), where the planar chain needs no recursion:
//   sum_b W_ab (cos(th_a - th_b) al_b + sin(th_a - th_b) om_b^2)
//     = (tau - b qd)_a - (tau - b qd)_{a+1},
//   W_ab = l_a l_b sum_{i >= max(a, b)} m_i,
// and qdd_a = al_a - al_{a-1}.  Lane r of each 16-lane row owns link r and
// keeps row r of the mass matrix in registers; the other links' values reach
// it by lane reads, and the matrix is eliminated by Gauss-Jordan steps in the
// same registers (symmetric positive definite: no pivoting), so an evaluation
// of the dynamics has no LDS access and no barrier.  What bounds both kernels
// is the chain of dependent FP64 operations of one evaluation; the recursive
// Newton-Euler passes, Cholesky and substitutions through LDS that this
// replaced took 15 us per evaluation at 13 links (4 RK4 substeps 244 us,
// linearization 83 us); see the kernels for the present figures.
// Everything runs in FP64 (the model is tiny); outputs are written in the
// problem dtype.
#include <hip/hip_runtime.h>
#include <math.h>

#include "internal.hpp"

namespace empc {

namespace {

// 1 / x by the hardware estimate and two Newton steps (the estimate's
// relative error of about 2^-23 is squared twice): within 1-2 units in the
// last place, an eighth of the dependent instructions of a division.
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// Link r's part of the chain, r = lane mod 16 (every 16-lane row alike).
// NB >= N: compile-time row length; links past N have W = 0 and a unit
// diagonal, so they never couple to the others.
template <int NB>
struct Link {
    int r;
    bool in;       // r < N
    double W[NB];  // l_r l_k sum of the masses from link max(r, k) on
    double b;      // viscous damping (0 past N)

    template <typename T>
    __device__ __forceinline__ void load(int N, const T *mass, const T *len, double damping) {
        r = threadIdx.x & 15;
        in = r < N;
        const double l = in ? (double)len[r] : 0.0;
        const double mu = row_scan_down<double>(in ? (double)mass[r] : 0.0);
        b = in ? damping : 0.0;
#pragma unroll
        for (int k = 0; k < NB; ++k)
            W[k] = l * lane_bcast<double>(l, k) * (k > r ? lane_bcast<double>(mu, k) : mu);
    }
    // torque on the absolute angle: t_r - t_{r+1} with t = tau - b qd
    __device__ __forceinline__ double torque(double tau, double om) const {
        const double t = in ? tau - b * (om - row_shift_up<double>(om, 1)) : 0.0;
        return t - row_shift_down<double>(t, 1);
    }
    // row r of the mass matrix and the centripetal sum sum_k W sin om_k^2
    __device__ __forceinline__ double row(double th, double om, double *a) const {
        double s, c;
        sincos(th, &s, &c);
        const double o2 = om * om;
        double h = 0.0;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const double ck = lane_bcast<double>(c, k), sk = lane_bcast<double>(s, k);
            a[k] = W[k] * (c * ck + s * sk);
            h += W[k] * (s * ck - c * sk) * lane_bcast<double>(o2, k);
            if (k == r && !in) a[k] = 1.0;
        }
        return h;
    }
    // absolute accelerations: Gauss-Jordan on (mass matrix | torque)
    __device__ __forceinline__ double acceleration(double th, double om, double tau) const {
        double a[NB];
        double y = torque(tau, om);
        y -= row(th, om, a);
        double own = 0.0;  // reciprocal of this row's pivot
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const double ip = recip(lane_bcast<double>(a[j], j));
            const double f = r == j ? 0.0 : a[j] * ip;
            own = r == j ? ip : own;
#pragma unroll
            for (int k = j + 1; k < NB; ++k) a[k] -= f * lane_bcast<double>(a[k], j);
            y -= f * lane_bcast<double>(y, j);
        }
        return y * own;
    }
};

// ---------------------------------------------------------------------------
// Linearization.  Eight wavefronts: the first three each run the dynamics
// (the same values) and build one of the right-hand sides' blocks, the rest
// is 32 x 32 matrix products on the FP64 matrix cores, a 16 x 16 tile of a
// product per wavefront, two products at a time.
constexpr int LIN_THREADS = 512;
constexpr int LDM = 34;             // row stride of the 32 x 32 matrices in LDS
constexpr int MSZ = 32 * LDM;
constexpr int LDR = 50;             // row stride of the right-hand sides [16][48]
constexpr int HOLD_BLOCKS = 4;      // blocks of four terms above the leading three

typedef double v4d __attribute__((ext_vector_type(4)));

// 1 / (k + 1)!, k = 0..18
__device__ constexpr double hold_coef(int k) {
    double f = 1.0;
    for (int i = 2; i <= k + 1; ++i) f *= (double)i;
    return 1.0 / f;
}

// 13 links: 83 us with recursive dual-number passes and VALU products,
// 16 us in this form (error of A_d, B_d, w_d against 64-bit references: 1.3e-13
// before, 1.1e-14 now, FP64 robot).
template <typename T, int NB>
__global__ __launch_bounds__(LIN_THREADS) void nlink_linearize_kernel(
    int N, const T *__restrict__ mass_in, const T *__restrict__ len_in, double b, double dt,
    const T *__restrict__ x_in, const T *__restrict__ u_in, T *__restrict__ Ad,
    T *__restrict__ Bd, T *__restrict__ wd) {
    // Y = A h and its powers; H: the right-hand sides, then the polynomial;
    // F: [B | w].  Rows and columns past n stay zero.
    __shared__ double Y[MSZ], Y2[MSZ], Y3[MSZ], Y4[MSZ], H[MSZ], F[MSZ];
    __shared__ double qdd[16], dotp[3][16], colsum[32];
    static_assert(16 * LDR <= MSZ, "right-hand sides fit");
    const int tid = threadIdx.x, n = 2 * N, m = N;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    double iv[NB];  // row r of dqdd / d(torque on the absolute angles)
    double xs = 0.0;  // this lane's column entry of (q, qd, tau) for the offset
    if (wave < 3) {
        Link<NB> L;
        L.load(N, mass_in, len_in, b);
        const int r = L.r;
        const double q = L.in ? (double)x_in[r] : 0.0, qd = L.in ? (double)x_in[N + r] : 0.0;
        const double u = L.in ? (double)u_in[r] : 0.0;
        xs = wave == 0 ? q : wave == 1 ? qd : u;
        const double th = row_scan_up<double>(q), om = row_scan_up<double>(qd);
        double s, c;
        sincos(th, &s, &c);
        double a[NB];
        double y = L.torque(u, om);
        y -= L.row(th, om, a);
        // in-place Gauss-Jordan inverse; each row is scaled by its pivot last
        double own = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const double ip = recip(lane_bcast<double>(a[j], j));
            const double f = r == j ? 0.0 : a[j] * ip;
            own = r == j ? ip : own;
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (k != j) a[k] -= f * lane_bcast<double>(a[k], j);
            a[j] = r == j ? 1.0 : -f;
        }
        double al = 0.0;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            a[k] *= own;
            al += a[k] * lane_bcast<double>(y, k);
        }
        // rows of differences: al_r - al_{r-1} = qdd_r
#pragma unroll
        for (int k = 0; k < NB; ++k) iv[k] = a[k] - row_shift_up<double>(a[k], 1);
        const double qa = al - row_shift_up<double>(al, 1);
        if (wave == 0 && grp == 0) qdd[r] = qa;
        // Row r of the right-hand sides of M dal/d(.) = ..., in the relative
        // coordinates.  With D_ab = W_ab (cos om_b^2 - sin al_b):
        //  q_s:  -sum_{c < s} D_ac for s <= a, sum_{c >= s} D_ac above;
        //  qd_s: -sum_{c >= s} 2 W_ac sin om_c, and the damping of joint s;
        //  tau_s: the unit torque of joint s.
        double e[NB];
        const double o2 = om * om;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const double ck = lane_bcast<double>(c, k), sk = lane_bcast<double>(s, k);
            const double sn = s * ck - c * sk, cs = c * ck + s * sk;
            e[k] = wave == 0 ? L.W[k] * (cs * lane_bcast<double>(o2, k) -
                                         sn * lane_bcast<double>(al, k))
                             : -2.0 * L.W[k] * sn * lane_bcast<double>(om, k);
        }
        double pre[NB];  // sums over c < s
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            pre[k] = t;
            t += e[k];
        }
        t = 0.0;
#pragma unroll
        for (int k = NB - 1; k >= 0; --k) {
            t += e[k];  // sum over c >= k
            const double unit = L.in ? (k == r ? 1.0 : k == r + 1 && k < N ? -1.0 : 0.0) : 0.0;
            const double v = wave == 0 ? (k <= r ? -pre[k] : t)
                                       : wave == 1 ? t - L.b * unit : unit;
            if (grp == 0) H[r * LDR + 16 * wave + k] = v;
        }
    } else {
        // the other wavefronts clear the matrices
        for (int e = tid - 192; e < MSZ; e += LIN_THREADS - 192)
            Y[e] = Y2[e] = Y3[e] = Y4[e] = F[e] = 0.0;
    }
    __syncthreads();
    // J block of wavefront w < 3: (rows of differences) x (its right-hand
    // sides), 16 x 16; row i is qdd_i, column s the s-th q, qd or tau
    if (wave < 3) {
        v4d acc = {0, 0, 0, 0};
#pragma unroll
        for (int k0 = 0; k0 < 16; k0 += 4) {
            double av = 0.0;
#pragma unroll
            for (int g = 0; g < 4; ++g)
                if (k0 + g < NB) av = grp == g ? iv[k0 + g < NB ? k0 + g : 0] : av;
            const double bv = k0 + grp < NB && col < NB ? H[(k0 + grp) * LDR + 16 * wave + col]
                                                        : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
        }
        double *to = wave == 2 ? F : Y;
        const int c0 = wave == 1 ? N : 0;
        const double scale = wave == 2 ? 1.0 : dt;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = grp + 4 * v;
            if (i < N && col < N) to[(N + i) * LDM + c0 + col] = acc[v] * scale;
            const double d = row_scan_up<double>(acc[v] * xs);  // lane 15 of the row: the sum
            if (col == 15) dotp[wave][i] = d;
        }
    } else if (wave == 3) {
        if (lane < N) Y[lane * LDM + N + lane] = dt;  // position rows of A: qd
    }
    __syncthreads();
    // f(x, u) ~ f0 + A (x' - x) + B (u' - u): A = [[0, I], [Jq, Jqd]],
    // B = [[0], [Ju]], offset w = f0 - A x - B u (position rows: 0)
    if (tid < N) F[(N + tid) * LDM + m] = qdd[tid] - (dotp[0][tid] + dotp[1][tid] + dotp[2][tid]);
    if (tid >= 64 && tid < 96) {
        double cs = 0.0;
        for (int i = 0; i < n; ++i) cs += fabs(Y[i * LDM + tid - 64]);
        colsum[tid - 64] = cs;
    }
    __syncthreads();
    // Zero-order hold: Phi = exp(A dt), Gamma = int_0^dt exp(A s) ds, then
    // A_d = Phi, [B_d w_d] = Gamma [B w].  Scaling and squaring on h = dt /
    // 2^sc with |A h|_1 <= 1: G = sum_{k <= 18} (A h)^k / (k+1)! (truncation
    // below 1e-18) in blocks of four powers (Paterson-Stockmeyer: 7 products
    // where Horner takes 18), Phi(h) = I + A h G, V = h G [B w]; each
    // squaring V <- V + Phi V, Phi <- Phi Phi.
    double cmax = colsum[lane & 31];
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) cmax = fmax(cmax, __shfl_xor(cmax, o, 64));
    int sc = 0;
    while (cmax > 1.0 && sc < 66) {
        cmax *= 0.5;
        ++sc;
    }
    sc = __builtin_amdgcn_readfirstlane(sc);
    const double scl = ldexp(1.0, -sc), h = dt * scl;
    for (int e = tid; e < MSZ; e += LIN_THREADS) Y[e] *= scl;
    __syncthreads();
    const int prod = wave >> 2, ti = (wave >> 1) & 1, tj = wave & 1;
    const bool live = 16 * ti < n && 16 * tj < n;  // tiles past the states stay zero
    // this wavefront's tile of A B: lane holds rows 16 ti + grp + 4 v, column
    // 16 tj + col
    auto product = [&](const double *A, const double *B) {
        v4d acc = {0, 0, 0, 0};
        if (live) {
            const double *ap = A + (16 * ti + col) * LDM + grp, *bp = B + grp * LDM + 16 * tj + col;
            for (int k0 = 0; k0 < n; k0 += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[k0], bp[k0 * LDM], acc, 0, 0, 0);
        }
        return acc;
    };
    const int e0 = (16 * ti + grp) * LDM + 16 * tj + col;  // element of v: + 4 v LDM
    auto store = [&](double *to, v4d x) {
        if (live) {
#pragma unroll
            for (int v = 0; v < 4; ++v) to[e0 + 4 * v * LDM] = x[v];
        }
    };
    auto eye = [&](int v) {
        const int i = 16 * ti + grp + 4 * v;
        return i == 16 * tj + col && i < n ? 1.0 : 0.0;
    };
    if (prod == 0) store(Y2, product(Y, Y));
    __syncthreads();
    if (prod == 0)
        store(Y3, product(Y2, Y));
    else
        store(Y4, product(Y2, Y2));
    // H = c16 I + c17 Y + c18 Y^2 (its right-hand sides have been read)
    if (prod == 0) {
        v4d x = {0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < 4; ++v)
            x[v] = hold_coef(16) * eye(v) + hold_coef(17) * Y[e0 + 4 * v * LDM] +
                   hold_coef(18) * Y2[e0 + 4 * v * LDM];
#pragma unroll
        for (int v = 0; v < 4; ++v) H[e0 + 4 * v * LDM] = x[v];
    }
    __syncthreads();
#pragma unroll
    for (int blk = HOLD_BLOCKS - 1; blk >= 0; --blk) {  // H <- H Y^4 + block
        v4d x = {0, 0, 0, 0};
        if (prod == 0) {
            x = product(H, Y4);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] += hold_coef(4 * blk) * eye(v) + hold_coef(4 * blk + 1) * Y[e0 + 4 * v * LDM] +
                        hold_coef(4 * blk + 2) * Y2[e0 + 4 * v * LDM] +
                        hold_coef(4 * blk + 3) * Y3[e0 + 4 * v * LDM];
        }
        __syncthreads();
        if (prod == 0) store(H, x);
        __syncthreads();
    }
    double *Ph = Y2, *V = Y3;  // the powers are no longer needed
    {
        v4d x = prod == 0 ? product(Y, H) : product(H, F);
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = prod == 0 ? x[v] + eye(v) : h * x[v];
        __syncthreads();
        store(prod == 0 ? Ph : V, x);
        __syncthreads();
    }
    for (int s = 0; s < sc; ++s) {
        v4d x = product(Ph, prod == 0 ? Ph : V);
        if (prod == 1) {
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] += V[e0 + 4 * v * LDM];
        }
        __syncthreads();
        store(prod == 0 ? Ph : V, x);
        __syncthreads();
    }
    for (int e = tid; e < n * 32; e += LIN_THREADS) {
        const int i = e / 32, j = e % 32;
        if (j < n) Ad[i * n + j] = (T)Ph[i * LDM + j];
        if (j < m) Bd[i * m + j] = (T)V[i * LDM + j];
        if (j == m) wd[i] = (T)V[i * LDM + j];
    }
}

constexpr int STEP_THREADS = 64;

// Classical RK4 over dt in `sub` substeps, tau held; one wavefront (its four
// 16-lane rows compute the same values).  The increments of the absolute
// angles and rates are accumulated and turned back into relative ones at
// the end.  13 links, 4 substeps: 244 us -> 31 us, 1.9 us per evaluation of
// the dynamics.
template <typename T, int NB>
__global__ __launch_bounds__(STEP_THREADS) void nlink_step_kernel(
    int N, const T *__restrict__ mass_in, const T *__restrict__ len_in, double b, double dt,
    int sub, const T *x_in, const T *__restrict__ u_in, T *x_out) {
    Link<NB> L;
    L.load(N, mass_in, len_in, b);
    const double tau = L.in ? (double)u_in[L.r] : 0.0;
    const double q = L.in ? (double)x_in[L.r] : 0.0, qd = L.in ? (double)x_in[N + L.r] : 0.0;
    const double th0 = row_scan_up<double>(q), om0 = row_scan_up<double>(qd);
    double dth = 0.0, dom = 0.0;
    const double hs = dt / sub;
    for (int s = 0; s < sub; ++s) {
        double ath = 0.0, aom = 0.0, oth = dth, oom = dom;
        // the four stages share one inlined copy of the dynamics; weights
        // 1, 2, 2, 1 and next-stage offsets 0.5, 0.5, 1
#pragma unroll 1
        for (int stage = 0; stage < 4; ++stage) {
            const double th = th0 + oth, kth = om0 + oom;
            const double kom = L.acceleration(th, kth, tau);
            const double w = stage == 0 || stage == 3 ? 1.0 : 2.0;
            ath += w * kth;
            aom += w * kom;
            const double off = (stage == 2 ? 1.0 : 0.5) * hs;
            oth = dth + off * kth;
            oom = dom + off * kom;
        }
        dth += hs / 6.0 * ath;
        dom += hs / 6.0 * aom;
    }
    const double nq = q + (dth - row_shift_up<double>(dth, 1));
    const double nqd = qd + (dom - row_shift_up<double>(dom, 1));
    if (threadIdx.x < 16 && L.in) {
        x_out[L.r] = (T)nq;
        x_out[N + L.r] = (T)nqd;
    }
}

// instance of the smallest even row length that holds N links
template <typename F>
hipError_t by_links(int N, F &&go) {
    switch ((N + 1) / 2) {
        case 1: return go(std::integral_constant<int, 2>());
        case 2: return go(std::integral_constant<int, 4>());
        case 3: return go(std::integral_constant<int, 6>());
        case 4: return go(std::integral_constant<int, 8>());
        case 5: return go(std::integral_constant<int, 10>());
        case 6: return go(std::integral_constant<int, 12>());
        case 7: return go(std::integral_constant<int, 14>());
        default: return go(std::integral_constant<int, 16>());
    }
}

}  // namespace

template <typename T>
hipError_t launch_nlink_linearize(int N, const T *mass, const T *len, double b, double dt,
                                  const T *x, const T *u, T *Ad, T *Bd, T *wd, hipStream_t s) {
    return by_links(N, [&](auto nb) {
        hipLaunchKernelGGL((nlink_linearize_kernel<T, decltype(nb)::value>), dim3(1),
                           dim3(LIN_THREADS), 0, s, N, mass, len, b, dt, x, u, Ad, Bd, wd);
        return hipGetLastError();
    });
}
template <typename T>
hipError_t launch_nlink_step(int N, const T *mass, const T *len, double b, double dt, int sub,
                             const T *x, const T *u, T *x_next, hipStream_t s) {
    return by_links(N, [&](auto nb) {
        hipLaunchKernelGGL((nlink_step_kernel<T, decltype(nb)::value>), dim3(1),
                           dim3(STEP_THREADS), 0, s, N, mass, len, b, dt, sub, x, u, x_next);
        return hipGetLastError();
    });
}
template hipError_t launch_nlink_linearize<float>(int, const float *, const float *, double,
                                                  double, const float *, const float *, float *,
                                                  float *, float *, hipStream_t);
template hipError_t launch_nlink_linearize<double>(int, const double *, const double *, double,
                                                   double, const double *, const double *,
                                                   double *, double *, double *, hipStream_t);
template hipError_t launch_nlink_step<float>(int, const float *, const float *, double, double, int,
                                             const float *, const float *, float *, hipStream_t);
template hipError_t launch_nlink_step<double>(int, const double *, const double *, double, double,
                                              int, const double *, const double *, double *,
                                              hipStream_t);

}  // namespace empc

using namespace empc;

empc_status empc_fail_internal(empc_status s, const char *msg);

namespace {

empc_status check_robot(const empc_nlink *R, double dt) {
    if (!R) return empc_fail_internal(EMPC_EINVAL, "robot is NULL");
    if (R->dtype != EMPC_F32 && R->dtype != EMPC_F64)
        return empc_fail_internal(EMPC_EINVAL, "unknown dtype");
    if (R->links < 1) return empc_fail_internal(EMPC_EINVAL, "links must be >= 1");
    if (R->links > NLINK_MAX)
        return empc_fail_internal(EMPC_EUNSUPPORTED, "more links than the library supports (16)");
    if (!R->mass || !R->length) return empc_fail_internal(EMPC_EINVAL, "mass and length are required");
    if (!isfinite(R->damping)) return empc_fail_internal(EMPC_EINVAL, "damping must be finite");
    if (!(dt > 0.0) || !isfinite(dt)) return empc_fail_internal(EMPC_EINVAL, "dt must be finite and > 0");
    return EMPC_OK;
}

empc_status launched(hipError_t e) {
    if (e == hipSuccess) return EMPC_OK;
    return empc_fail_internal(EMPC_EDEVICE, hipGetErrorString(e));
}

}  // namespace

extern "C" {

empc_status empc_nlink_linearize(const empc_nlink *robot, double dt, const void *x,
                                 const void *u, void *Ad, void *Bd, void *wd, void *stream) {
    empc_status st = check_robot(robot, dt);
    if (st) return st;
    if (!x || !u || !Ad || !Bd || !wd)
        return empc_fail_internal(EMPC_EINVAL, "x, u, Ad, Bd and wd are required");
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return launched(e);
    hipStream_t s = (hipStream_t)stream;
    const int N = robot->links;
    if (robot->dtype == EMPC_F32)
        e = launch_nlink_linearize<float>(N, (const float *)robot->mass, (const float *)robot->length,
                                          robot->damping, dt, (const float *)x, (const float *)u,
                                          (float *)Ad, (float *)Bd, (float *)wd, s);
    else
        e = launch_nlink_linearize<double>(N, (const double *)robot->mass,
                                           (const double *)robot->length, robot->damping, dt,
                                           (const double *)x, (const double *)u, (double *)Ad,
                                           (double *)Bd, (double *)wd, s);
    return launched(e);
}

empc_status empc_nlink_step(const empc_nlink *robot, double dt, int32_t substeps, const void *x,
                            const void *u, void *x_next, void *stream) {
    empc_status st = check_robot(robot, dt);
    if (st) return st;
    if (substeps < 1 || substeps > 1000000)
        return empc_fail_internal(EMPC_EINVAL, "substeps outside [1, 10^6]");
    if (!x || !u || !x_next) return empc_fail_internal(EMPC_EINVAL, "x, u and x_next are required");
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return launched(e);
    hipStream_t s = (hipStream_t)stream;
    const int N = robot->links;
    if (robot->dtype == EMPC_F32)
        e = launch_nlink_step<float>(N, (const float *)robot->mass, (const float *)robot->length,
                                     robot->damping, dt, substeps, (const float *)x,
                                     (const float *)u, (float *)x_next, s);
    else
        e = launch_nlink_step<double>(N, (const double *)robot->mass, (const double *)robot->length,
                                      robot->damping, dt, substeps, (const double *)x,
                                      (const double *)u, (double *)x_next, s);
    return launched(e);
}

}  // extern "C"
