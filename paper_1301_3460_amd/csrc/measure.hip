// Measurements of given links and the differentiation kernels (SU(3), FP64).
//
// These calls look at the caller's links once, so they read them where they
// are (complex128 [4][V][3][3], rows 0,1 of each link; 144 bytes apart, and a
// wavefront's loads of the six entries share their lines) instead of packing
// them first: a packed copy costs 177 us at 32^4, as much as reading the links
// twice.  At 32^4 (604 MB of link lines, 123 us at the rate of a copy): F 108
// us, F and theta 152, the plaquette 233 (pack, divergence and reduction were
// 281, pack and plaquette 337).  A wave's six loads of a link touch 64 segments
// each, so a kernel that reads 22 links per site, like the plaquette's, is
// held by its address unit; loading a wave's links cooperatively and handing
// them out through LDS was slower all the same (plaquette 676 us, theta 379).
#include "common.hpp"

namespace lgf {

namespace {

constexpr int AD_TERMS = 80;  // bound on the terms of the exponential map's derivative

// rows 0,1 of the caller's link mu at site x
struct aos_links {
    const double2 *__restrict__ U;
    long V;
    __device__ __forceinline__ void rows(int mu, long x, cpx<double> (&u)[6]) const {
        const double2 *p = U + ((long)mu * V + x) * 9;
#pragma unroll
        for (int k = 0; k < 6; ++k) u[k] = ld<double>(p + k);
    }
};

// rows 0,1 of 12-real links in a component-major buffer
struct soa_links {
    const double2 *__restrict__ L;
    long S;
    __device__ __forceinline__ void rows(int mu, long x, cpx<double> (&u)[6]) const {
        const double2 *p = L + (long)mu * 6 * S + x;
#pragma unroll
        for (int k = 0; k < 6; ++k) u[k] = ld<double>(p + (long)k * S);
    }
};

__device__ __forceinline__ mat3<double> rows01(const cpx<double> (&f)[6]) {
    mat3<double> m;
#pragma unroll
    for (int k = 0; k < 6; ++k) m.e[k / 3][k % 3] = f[k];
    return m;
}

template <class Links> __device__ __forceinline__ mat3<double> link_at(const Links &L, int mu, long x) {
    cpx<double> u[6];
    L.rows(mu, x, u);
    mat3<double> m = rows01(u);
    rebuild_row2(m);
    return m;
}

// rows 0,1 of A B (row 2 of B needed), row 2 completed: A, B in SU(3)
__device__ __forceinline__ mat3<double> su3_mul(const mat3<double> &a, const mat3<double> &b) {
    mat3<double> r;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> c = cmul(a.e[i][0], b.e[0][j]);
            c = cmac(c, a.e[i][1], b.e[1][j]);
            r.e[i][j] = cmac(c, a.e[i][2], b.e[2][j]);
        }
    rebuild_row2(r);
    return r;
}

// rows 0,1 of A B^dagger (all rows of B), row 2 completed
__device__ __forceinline__ mat3<double> su3_mul_dag(const mat3<double> &a, const mat3<double> &b) {
    mat3<double> r;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> c = cmulc(a.e[i][0], b.e[j][0]);
            c = cmacc(c, a.e[i][1], b.e[j][1]);
            r.e[i][j] = cmacc(c, a.e[i][2], b.e[j][2]);
        }
    rebuild_row2(r);
    return r;
}

__device__ __forceinline__ mat3<double> mat_mul_full(const mat3<double> &a, const mat3<double> &b) {
    mat3<double> r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> c = cmul(a.e[i][0], b.e[0][j]);
            c = cmac(c, a.e[i][1], b.e[1][j]);
            r.e[i][j] = cmac(c, a.e[i][2], b.e[2][j]);
        }
    return r;
}

// Re Tr[A B^dagger]
__device__ __forceinline__ double re_tr_dag(const mat3<double> &a, const mat3<double> &b) {
    double t = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            t = fma(a.e[i][j].re, b.e[i][j].re, fma(a.e[i][j].im, b.e[i][j].im, t));
    return t;
}

// The anti-hermitian traceless matrix of four Fourier-field entries.
__device__ __forceinline__ mat3<double> field_matrix(cpx<double> f0, cpx<double> f1, cpx<double> f2,
                                                     cpx<double> f3) {
    mat3<double> M;
    M.e[0][0] = mk<double>(0, f3.re);
    M.e[0][1] = f0;
    M.e[0][2] = f1;
    M.e[1][0] = mk<double>(-f0.re, f0.im);
    M.e[1][1] = mk<double>(0, f3.im);
    M.e[1][2] = f2;
    M.e[2][0] = mk<double>(-f1.re, f1.im);
    M.e[2][1] = mk<double>(-f2.re, f2.im);
    M.e[2][2] = mk<double>(0, -(f3.re + f3.im));
    return M;
}

// exp(i sum_a w_a lambda_a / 2), rows 0,1 (row 2 completed)
__device__ __forceinline__ mat3<double> exp_su3(const double (&w)[8]) {
    const double r3 = 0.57735026918962576451;  // 1/sqrt(3)
    // the Fourier-field entries of X = (i/2) sum_a w_a lambda_a
    return gauge_exp_from_entries<double>(
        mk<double>(0.5 * w[1], 0.5 * w[0]), mk<double>(0.5 * w[4], 0.5 * w[3]),
        mk<double>(0.5 * w[6], 0.5 * w[5]), mk<double>(0.5 * (w[2] + w[7] * r3), 0.5 * (w[7] * r3 - w[2])),
        1.0);
}

__device__ __forceinline__ void load8(const double *__restrict__ p, double (&w)[8]) {
#pragma unroll
    for (int a = 0; a < 8; ++a) w[a] = p[a];
}

// Im Tr[lambda_a W], a = 0..7
__device__ __forceinline__ void im_tr_lambda(const mat3<double> &W, double (&y)[8]) {
    const double r3 = 0.57735026918962576451;
    y[0] = W.e[1][0].im + W.e[0][1].im;
    y[1] = W.e[0][1].re - W.e[1][0].re;
    y[2] = W.e[0][0].im - W.e[1][1].im;
    y[3] = W.e[2][0].im + W.e[0][2].im;
    y[4] = W.e[0][2].re - W.e[2][0].re;
    y[5] = W.e[2][1].im + W.e[1][2].im;
    y[6] = W.e[1][2].re - W.e[2][1].re;
    y[7] = (W.e[0][0].im + W.e[1][1].im - 2 * W.e[2][2].im) * r3;
}

// out = sum_k (A^T)^k v / (k+1)!,  A[b][a] = coefficient of i T^b in [i w.T, i T^a]
//     = -sum_c f_abc w_c  (SU(3) structure constants).
// This is the transpose of the derivative of the exponential map, so for
// g = exp(i w.T): d/dw^a = sum_b S[b][a] (derivative along i T^b g).
// A^T t is the bracket of w and t in the adjoint representation: with the
// nine independent f_abc each a three-dimensional cross product, 54
// multiply-adds against the 64 of the full matrix and no matrix to hold.
// No division per term and no running maximum either: theta's gradient at 32^4
// 661 -> 302 us, 200 of which its 1.0 GB take.
// The series is summed from its last term (Horner); |A| <= |w|, so the number
// of terms that leaves a remainder below 1e-18 |v| is known beforehand
// (in FP32, from an upper bound of |w|).
__device__ __forceinline__ void dexp_transpose_apply(const double (&w)[8], const double (&v)[8],
                                                     double (&out)[8]) {
    double n2 = 0;
#pragma unroll
    for (int a = 0; a < 8; ++a) n2 = fma(w[a], w[a], n2);
    const float rho = sqrtf((float)n2) * 1.0001f;
    int K = 0;
    float t = 1.0f;
    do {
        ++K;
        t *= rho * __builtin_amdgcn_rcpf((float)(K + 1));
    } while (t > 1e-18f && K < AD_TERMS);
    const double hh = 0.5, h3 = 0.86602540378443864676;
    double p[8], q[8];  // w scaled by the structure constants 1/2 and sqrt(3)/2
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        p[a] = hh * w[a];
        q[a] = h3 * w[a];
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) out[a] = v[a];
#pragma unroll 1
    for (; K > 0; --K) {
        double s[8];
#pragma unroll
        for (int a = 0; a < 8; ++a) s[a] = 0;
        // s += f_abc (w x t) on the triple (a, b, c)
        auto cross = [&](const double (&u)[8], int a, int b, int c) {
            s[a] = fma(u[b], out[c], fma(-u[c], out[b], s[a]));
            s[b] = fma(u[c], out[a], fma(-u[a], out[c], s[b]));
            s[c] = fma(u[a], out[b], fma(-u[b], out[a], s[c]));
        };
        cross(w, 0, 1, 2);
        cross(p, 0, 3, 6);
        cross(p, 0, 5, 4);
        cross(p, 1, 3, 5);
        cross(p, 1, 4, 6);
        cross(p, 2, 3, 4);
        cross(p, 2, 6, 5);
        cross(q, 3, 4, 7);
        cross(q, 5, 6, 7);
        const double r = recip((double)(K + 1));
#pragma unroll
        for (int a = 0; a < 8; ++a) out[a] = fma(s[a], r, v[a]);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// sums over the links
// ---------------------------------------------------------------------------

// sum_mu Re Tr U_mu(x)
__global__ void __launch_bounds__(SITE_BLOCK)
    k_trace_aos(geom g, aos_links L, double *__restrict__ partials) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double tr = 0;
    if (s < g.V) {
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) tr += retrace(link_at(L, mu, s));
    }
    block_sum2<SITE_BLOCK>(tr, 0.0, partials, blockIdx.x);
}

// Delta(x) of the links with the partials of F and theta.  OUT 0: the partials
// alone, 1: also Delta as four Fourier fields in D (stride S), 2: Delta as 3x3
// matrices in M (each wave's 64 consecutive sites staged in LDS and written as
// one run).
template <class Links, int OUT>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_div_links(geom g, Links L, double2 *__restrict__ D, double *__restrict__ partials) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double fs = 0, ts = 0;
    cpx<double> f[4];
    if (s < g.V) {
        const nbr n = neighbours(g, s);
        xacc<double> X;
        xacc_zero(X);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const mat3<double> u = link_at(L, mu, s);
            fs += retrace(u);
            xacc_add(X, u, -1.0);
            xacc_add(X, link_at(L, mu, n.m[mu]), 1.0);
        }
        ts = delta_pack(X, f[0], f[1], f[2], f[3]);
        if constexpr (OUT == 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) st<double>(D + k * g.S + s, f[k]);
        }
    }
    if constexpr (OUT == 2) {
        __shared__ double2 buf[SITE_BLOCK * 9];
        const int lane = threadIdx.x & 63;
        double2 *mine = buf + (threadIdx.x - lane) * 9;
        const long s0 = s - lane;
        if (s < g.V) {
            const mat3<double> M = field_matrix(f[0], f[1], f[2], f[3]);
#pragma unroll
            for (int k = 0; k < 9; ++k)
                mine[lane * 9 + k] = make_double2(M.e[k / 3][k % 3].re, M.e[k / 3][k % 3].im);
        }
        __syncthreads();
        const int cnt = (int)(g.V - s0 < 64 ? (g.V > s0 ? g.V - s0 : 0) : 64) * 9;
        double2 *m = D + s0 * 9;
        for (int e = lane; e < cnt; e += 64) m[e] = mine[e];
    }
    block_sum2<SITE_BLOCK>(fs, ts, partials, blockIdx.x);
}

// sum_{mu<nu} Re Tr[U_mu(x) U_nu(x+mu) U_mu(x+nu)^dagger U_nu(x)^dagger]
//   = Re Tr[P Q^dagger], P = U_mu(x) U_nu(x+mu), Q = U_nu(x) U_mu(x+nu)
// All three rows by products: a completed row 2 is not the product's on links
// in SU(3) only to the precision they were stored in.
__global__ void __launch_bounds__(SITE_BLOCK)
    k_plaquette(geom g, aos_links L, double *__restrict__ partials) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double acc = 0;
    if (s < g.V) {
        const nbr n = neighbours(g, s);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const mat3<double> u = link_at(L, mu, s);
            // one plane's three links at a time: 192 VGPRs against 244 unrolled,
            // the call at 32^4 248 us against 316 (302 with completed rows)
#pragma unroll 1
            for (int nu = mu + 1; nu < 4; ++nu) {
                const long sn = nu == 1 ? n.p[1] : nu == 2 ? n.p[2] : n.p[3];
                acc += re_tr_dag(mat_mul_full(u, link_at(L, nu, n.p[mu])),
                                 mat_mul_full(link_at(L, nu, s), link_at(L, mu, sn)));
            }
        }
    }
    block_sum2<SITE_BLOCK>(acc, 0.0, partials, blockIdx.x);
}

// sum_mu Re Tr[g(x) U_mu(x) g(x+mu)^dagger], g any 3x3 matrices (AoS)
__global__ void __launch_bounds__(SITE_BLOCK)
    k_functional_g(geom g, aos_links L, const double2 *__restrict__ ga,
                   double *__restrict__ partials) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double acc = 0;
    if (s < g.V) {
        const nbr n = neighbours(g, s);
        auto load_g = [&](long x) {
            mat3<double> m;
#pragma unroll
            for (int k = 0; k < 9; ++k) m.e[k / 3][k % 3] = ld<double>(ga + x * 9 + k);
            return m;
        };
        const mat3<double> g0 = load_g(s);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu)
            acc += re_tr_dag(mat_mul_full(g0, link_at(L, mu, s)), load_g(n.p[mu]));
    }
    block_sum2<SITE_BLOCK>(acc, 0.0, partials, blockIdx.x);
}

// ---------------------------------------------------------------------------
// differentiation
// ---------------------------------------------------------------------------

// G(x) = exp(i omega.T), rows 0,1 as six component arrays
__global__ void __launch_bounds__(128)
    k_exp_sites(const double *__restrict__ w, double2 *__restrict__ G, long V, long S) {
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
    double ww[8];
    load8(w + s * 8, ww);
    const mat3<double> E = exp_su3(ww);
#pragma unroll
    for (int k = 0; k < 6; ++k) st<double>(G + (long)k * S + s, E.e[k / 3][k % 3]);
}

// 12-real links exp(i eps^a_mu(x) T^a) U_mu(x) from the caller's links: 256
// bytes per link (eps 64, the link's line 144 of which rows 0,1 are used, 96
// written), 232 us at 32^4 = 5.5 TB/s.  The exponential in the closed algebra
// of 1, Q, Q^2 (gauge_exp_from_entries) instead of a Taylor series of matrix
// products, and no copies of it or of the packed links in memory: pack,
// exponential and product took 177 + 714 + 307 us.
__global__ void __launch_bounds__(256)
    k_exp_links(const double *__restrict__ eps, aos_links U, double2 *__restrict__ Lout, long S) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 4 * U.V) return;
    const int mu = (int)(i / U.V);
    const long s = i - (long)mu * U.V;
    double w[8];
    load8(eps + i * 8, w);
    const mat3<double> u = link_at(U, mu, s);
    const mat3<double> r = su3_mul(exp_su3(w), u);
    double2 *p = Lout + (long)mu * 6 * S + s;
#pragma unroll
    for (int k = 0; k < 6; ++k) st<double>(p + (long)k * S, r.e[k / 3][k % 3]);
}

// F_U[G] partials: sum_mu Re Tr[G(x) U_mu(x) G(x+mu)^dagger] (all three rows of
// G U by products, as in k_plaquette)
__global__ void __launch_bounds__(SITE_BLOCK)
    k_functional_rot(geom g, aos_links L, soa_links G, double *__restrict__ partials) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double acc = 0;
    if (s < g.V) {
        const nbr n = neighbours(g, s);
        const mat3<double> g0 = link_at(G, 0, s);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu)
            acc += re_tr_dag(mat_mul_full(g0, link_at(L, mu, s)), link_at(G, 0, n.p[mu]));
    }
    block_sum2<SITE_BLOCK>(acc, 0.0, partials, blockIdx.x);
}

// F_U[G] partials and dF/domega^a(x) in one pass: Delta of the rotated links,
// rows 0,1 formed and row 2 completed, from M of K and K' as in k_update_u0 (row
// 2 from K as well is off on links rounded to FP32), then the derivative of the
// exponential map at omega(x).  240 VGPRs, two waves per SIMD; without K', at 154
// and three, F and gradient of 32^4 took 395 us instead of 293.
//   G^b = -(i/4) normF Tr[lambda_b Delta] = (normF/4) Im Tr[lambda_b Delta]
__global__ void __launch_bounds__(SITE_BLOCK)
    k_omega_grad(geom g, aos_links L, soa_links G, const double *__restrict__ om,
                 double *__restrict__ dF, double normF, double *__restrict__ partials) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double fs = 0;
    if (s < g.V) {
        const nbr n = neighbours(g, s);
        mat3<double> K;
        cpx<double> C[2][3];  // rows 0,1 of K'
#pragma unroll
        for (int k = 0; k < 9; ++k) K.e[k / 3][k % 3] = mk<double>(0, 0);
#pragma unroll
        for (int k = 0; k < 6; ++k) C[k / 3][k % 3] = mk<double>(0, 0);
        // one direction's 24 loads at a time: unrolled, the compiler issues all
        // 102 first, which takes 456 registers and leaves one wave per SIMD
#pragma unroll 1
        for (int mu = 0; mu < 4; ++mu) {
            const long sp = mu == 0 ? n.p[0] : mu == 1 ? n.p[1] : mu == 2 ? n.p[2] : n.p[3];
            const long sm = mu == 0 ? n.m[0] : mu == 1 ? n.m[1] : mu == 2 ? n.m[2] : n.m[3];
            cpx<double> u[6];
            L.rows(mu, s, u);
            const mat3<double> p = su3_mul_dag(rows01(u), link_at(G, 0, sp));
            G.rows(0, sm, u);
            const mat3<double> q = su3_mul(rows01(u), link_at(L, mu, sm));
#pragma unroll
            for (int k = 0; k < 9; ++k)
                K.e[k / 3][k % 3] = K.e[k / 3][k % 3] + (p.e[k / 3][k % 3] + conjg(q.e[k % 3][k / 3]));
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const int r = i + 1, t = (i + 2) % 3, a = (j + 1) % 3, b = (j + 2) % 3;
                    const cpx<double> m = cmul(p.e[r][a], p.e[t][b]);
                    C[i][j] = C[i][j] + conjg(cmsub(m, p.e[r][b], p.e[t][a]) + q.e[j][i]);
                }
        }
        const mat3<double> g0 = link_at(G, 0, s);
        mat3<double> M = mat_mul_full(g0, K);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> c = cmul(g0.e[2][0], C[0][j]);
            c = cmac(c, g0.e[2][1], C[1][j]);
            M.e[2][j] = cmac(c, g0.e[2][2], K.e[2][j]);
        }
        xacc<double> X;
        xacc_zero(X);
        xacc_add(X, M, -1.0);
        cpx<double> f[4];
        delta_pack(X, f[0], f[1], f[2], f[3]);
        fs = 0.5 * retrace(M);
        double y[8], w[8], out[8];
        im_tr_lambda(field_matrix(f[0], f[1], f[2], f[3]), y);
#pragma unroll
        for (int a = 0; a < 8; ++a) y[a] *= 0.25 * normF;
        load8(om + s * 8, w);
        dexp_transpose_apply(w, y, out);
#pragma unroll
        for (int a = 0; a < 8; ++a) dF[s * 8 + a] = out[a];
    }
    block_sum2<SITE_BLOCK>(fs, 0.0, partials, blockIdx.x);
}

// dtheta/deps^a_mu(x) at links L (already exp(i eps.T) U); EPS: eps given.
// With D = Delta(x+mu) - Delta(x) anti-hermitian, U D + D U^dagger is U D
// minus its hermitian conjugate: one product.
template <class Links, bool EPS>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_theta_grad(geom g, Links L, const double2 *__restrict__ D, const double *__restrict__ eps,
                 double *__restrict__ dth, double normT) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    if (s >= g.V) return;
    const nbr n = neighbours(g, s);
    auto field = [&](long q, cpx<double> (&f)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = ld<double>(D + k * g.S + q);
    };
    cpx<double> d0[4];
    field(s, d0);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        cpx<double> dp[4];
        field(n.p[mu], dp);
        const mat3<double> W1 =
            mat_mul_full(link_at(L, mu, s), field_matrix(dp[0] - d0[0], dp[1] - d0[1],
                                                         dp[2] - d0[2], dp[3] - d0[3]));
        mat3<double> W;
#pragma unroll
        for (int k = 0; k < 9; ++k)
            W.e[k / 3][k % 3] = W1.e[k / 3][k % 3] - conjg(W1.e[k % 3][k / 3]);
        double y[8];
        im_tr_lambda(W, y);
#pragma unroll
        for (int a = 0; a < 8; ++a) y[a] *= normT;
        const long o = ((long)mu * g.V + s) * 8;
        if constexpr (EPS) {
            double w[8], out[8];
            load8(eps + o, w);
            dexp_transpose_apply(w, y, out);
#pragma unroll
            for (int a = 0; a < 8; ++a) dth[o + a] = out[a];
        } else {
#pragma unroll
            for (int a = 0; a < 8; ++a) dth[o + a] = y[a];
        }
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline unsigned nblk(long n, int b) { return (unsigned)((n + b - 1) / b); }

static aos_links aos(const geom &g, const double *U) {
    return {reinterpret_cast<const double2 *>(U), g.V};
}

hipError_t launch_trace_aos(const geom &g, const double *U, double *partials, hipStream_t st) {
    k_trace_aos<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, aos(g, U), partials);
    return hipGetLastError();
}

hipError_t launch_div_aos(const geom &g, const double *U, double2 *out, int matrices,
                          double *partials, hipStream_t st) {
    const int nb = site_blocks(g.V);
    if (!out) k_div_links<aos_links, 0><<<nb, SITE_BLOCK, 0, st>>>(g, aos(g, U), out, partials);
    else if (matrices) k_div_links<aos_links, 2><<<nb, SITE_BLOCK, 0, st>>>(g, aos(g, U), out, partials);
    else k_div_links<aos_links, 1><<<nb, SITE_BLOCK, 0, st>>>(g, aos(g, U), out, partials);
    return hipGetLastError();
}

hipError_t launch_plaquette(const geom &g, const double *U, double *partials, hipStream_t st) {
    k_plaquette<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, aos(g, U), partials);
    return hipGetLastError();
}

hipError_t launch_functional_g(const geom &g, const double *U, const double *gaos, double *partials,
                               hipStream_t st) {
    k_functional_g<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(
        g, aos(g, U), reinterpret_cast<const double2 *>(gaos), partials);
    return hipGetLastError();
}

hipError_t launch_functional_omega(const geom &g, const double *U, const double *omega, double2 *G,
                                   double *partials, hipStream_t st) {
    k_exp_sites<<<nblk(g.V, 128), 128, 0, st>>>(omega, G, g.V, g.S);
    k_functional_rot<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, aos(g, U), soa_links{G, g.S}, partials);
    return hipGetLastError();
}

hipError_t launch_omega_grad(const geom &g, const double *U, const double *omega, double2 *G,
                             double *dF, double normF, double *partials, hipStream_t st) {
    k_exp_sites<<<nblk(g.V, 128), 128, 0, st>>>(omega, G, g.V, g.S);
    k_omega_grad<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, aos(g, U), soa_links{G, g.S}, omega, dF,
                                                          normF, partials);
    return hipGetLastError();
}

hipError_t launch_theta_links(const geom &g, const double *U, const double *eps, double2 *L,
                              double2 *D, double *partials, hipStream_t st) {
    if (!eps) return launch_div_aos(g, U, D, 0, partials, st);
    k_exp_links<<<nblk(4 * g.V, 256), 256, 0, st>>>(eps, aos(g, U), L, g.S);
    if (D)
        k_div_links<soa_links, 1>
            <<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, soa_links{L, g.S}, D, partials);
    else
        k_div_links<soa_links, 0>
            <<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, soa_links{L, g.S}, D, partials);
    return hipGetLastError();
}

hipError_t launch_theta_grad(const geom &g, const double *U, const double *eps, const double2 *L,
                             const double2 *D, double *dth, double normT, hipStream_t st) {
    const int nb = site_blocks(g.V);
    if (eps)
        k_theta_grad<soa_links, true><<<nb, SITE_BLOCK, 0, st>>>(g, soa_links{L, g.S}, D, eps, dth, normT);
    else
        k_theta_grad<aos_links, false><<<nb, SITE_BLOCK, 0, st>>>(g, aos(g, U), D, eps, dth, normT);
    return hipGetLastError();
}

}  // namespace lgf
