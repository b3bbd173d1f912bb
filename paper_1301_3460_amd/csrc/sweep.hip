// HIP kernels of the Fourier-accelerated Landau gauge-fixing sweep (gfx950).
//
// One sweep (one gauge update) is four launches plus a one-block finalize:
//   fft_xy(-1)  2D transform over the contiguous (x, y) planes, in place
//   fft_zt(0)   2D transform over (z, t), scaling by p2max/(V p2), inverse
//               (z, t) transform, in place: tiles of W consecutive xy-sites
//   fft_xy(+1)  inverse (x, y) transform -> L Delta
//   update      g = reunit(1 + alpha/2 L Delta) at x and its 8 neighbours,
//               U'_mu(x) = g(x) U_mu(x) g(x+mu)^dagger (written), and the next
//               Delta(x) from U'_mu(x) and the recomputed U'_mu(x-mu), with
//               block partial sums of F and theta
//   finalize    fixed-order sum of the partials, stopping test
// The form above stores the links of every sweep (double-buffered, as the
// update reads U_mu(x-mu) of other threads): SU(2), 8- and 18-real links and
// FP64 sweeps below 49152 sites.  The FP64 sweeps of larger lattices and the
// FP32 sweeps of an SU(3) mixed solve store no links: their inverse (x, y)
// pass (or k_gauge_acc after it) turns L Delta into G <- g G, double-buffered,
// and the update (k_update_u0, k_update_shared) forms G U0 G^dagger from the
// constant input copy U0; k_unpack_rotated writes them once, at the end.
// Small lattices run the four transforms of a field in one block (fft_small.hip),
// take a lane per link in the update (k_update_dirs) and finalize inside the
// next sweep's first kernel.
#include <type_traits>

#include "common.hpp"

namespace lgf {

// ---------------------------------------------------------------------------
// layout conversion
// ---------------------------------------------------------------------------

// A caller link (complex128 AoS, rows 0,1; all three rows for the 18-real
// format) as an SU(3) matrix of type T.
template <class T, int LF> __device__ __forceinline__ mat3<T> aos_link(const double2 *__restrict__ u) {
    constexpr int NIN = LF == 18 ? 9 : 6;
    mat3<T> m;
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
        const double2 v = u[k];
        m.e[k / 3][k % 3] = mk<T>((T)v.x, (T)v.y);
    }
    if constexpr (LF != 18) rebuild_row2(m);
    return m;
}

// complex128 [4][V][3][3] -> SoA of type T in link format LF
template <class T, int LF>
__global__ void __launch_bounds__(256) k_pack_links(const double2 *__restrict__ U,
                                                    vec2_t<T> *__restrict__ L, long V, long S) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 4 * V) return;
    const int mu = (int)(i / V);
    const long s = i - (long)mu * V;
    cpx<T> sl[LF / 2];
    link_to_slots<T, LF>(aos_link<T, LF>(U + i * 9), sl);
#pragma unroll
    for (int k = 0; k < LF / 2; ++k) st<T>(L + ((long)mu * (LF / 2) + k) * S + s, sl[k]);
}

template <int LF>
__global__ void __launch_bounds__(256) k_unpack_links(const double2 *__restrict__ L,
                                                      double2 *__restrict__ U, long V, long S) {
    // The block's 256 links are assembled in LDS and written out as one
    // contiguous run (consecutive lanes on consecutive 16-byte entries), not
    // as 144-byte strided pieces per lane.
    __shared__ double2 buf[256 * 9];
    const long i0 = (long)blockIdx.x * 256, i = i0 + threadIdx.x;
    const long n = min(4 * V - i0, 256L);
    if (i < 4 * V) {
        const int mu = (int)(i / V);
        const long s = i - (long)mu * V;
        const mat3<double> m = load_link<double, LF>(L, S, mu, s);
#pragma unroll
        for (int k = 0; k < 9; ++k)
            buf[threadIdx.x * 9 + k] = make_double2(m.e[k / 3][k % 3].re, m.e[k / 3][k % 3].im);
    }
    __syncthreads();
    double2 *u = U + i0 * 9;
    for (int e = threadIdx.x; e < n * 9; e += 256) u[e] = buf[e];
}

// anti-hermitian traceless matrix field (AoS 3x3 complex128) <-> 4 Fourier fields
__global__ void k_field_from_matrix(const double2 *__restrict__ M, double2 *__restrict__ D, long V,
                                    long S) {
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
    const double2 *m = M + s * 9;
    D[s] = m[1];
    D[S + s] = m[2];
    D[2 * S + s] = m[5];
    D[3 * S + s] = make_double2(m[0].y, m[4].y);
}

__global__ void k_matrix_from_field(const double2 *__restrict__ D, double2 *__restrict__ M, long V,
                                    long S) {
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
    const double2 f0 = D[s], f1 = D[S + s], f2 = D[2 * S + s], f3 = D[3 * S + s];
    double2 *m = M + s * 9;
    m[0] = make_double2(0.0, f3.x);
    m[1] = f0;
    m[2] = f1;
    m[3] = make_double2(-f0.x, f0.y);
    m[4] = make_double2(0.0, f3.y);
    m[5] = f2;
    m[6] = make_double2(-f1.x, f1.y);
    m[7] = make_double2(-f2.x, f2.y);
    m[8] = make_double2(0.0, -(f3.x + f3.y));
}

// ---------------------------------------------------------------------------
// finalize: fixed-order sum of block partials and the stopping test
// ---------------------------------------------------------------------------

constexpr int FIN_BLOCK = 1024;

// ---------------------------------------------------------------------------
// divergence and reductions of given links (first sweep of a solve)
// ---------------------------------------------------------------------------

// TF: real type of the Fourier field (T, or float for FP64 sweeps whose field
// is held in FP32)
// Delta(x) of the links link(mu, site), packed into the 4 field entries f;
// tr = sum_mu Re Tr U_mu(x); returns Tr[Delta Delta^dagger].
template <class T, class LinkFn>
__device__ __forceinline__ T divergence_at(const geom &g, long s, LinkFn link, cpx<T> (&f)[4],
                                           T &tr) {
    const nbr n = neighbours(g, s);
    xacc<T> X;
    xacc_zero(X);
    tr = 0;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        mat3<T> u = link(mu, s);
        tr += retrace(u);
        xacc_add(X, u, T(-1));
        mat3<T> um = link(mu, n.m[mu]);
        xacc_add(X, um, T(1));
    }
    return delta_pack(X, f[0], f[1], f[2], f[3]);
}

template <class T, class TF, int LF>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_div_reduce(geom g, const vec2_t<T> *__restrict__ L, vec2_t<TF> *__restrict__ D,
                 double *__restrict__ partials, const dev_status *__restrict__ status) {
    if (status->done) return;
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double fs = 0, ts = 0;
    if (s < g.V) {
        cpx<T> f[4];
        T tr;
        ts = (double)divergence_at<T>(
            g, s, [&](int mu, long x) { return load_link<T, LF>(L, g.S, mu, x); }, f, tr);
        fs = (double)tr;
#pragma unroll
        for (int k = 0; k < 4; ++k) st<TF>(D + k * g.S + s, cvt<TF>(f[k]));
    }
    block_sum2<SITE_BLOCK>(fs, ts, partials, blockIdx.x);
}

// ---------------------------------------------------------------------------
// fused update + next divergence
// ---------------------------------------------------------------------------

// GPRE: each site's transformation was computed beforehand and is read as
// rows 0,1 from GX (6 entries per site) instead of being formed from L Delta:
// g = exp((alpha/2) L Delta) of the exact step (k_gauge_exp), or the
// accumulated G of the FP32 sweeps (k_gauge_acc), whose links G U0 G^dagger
// come from the constant input copy U0 in Lin.  STORE: write the new links to
// Lout (the FP32 sweeps keep U0 and G instead).
template <class T, class TF, bool GPRE, int LF, bool STORE>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_update(geom g, const vec2_t<T> *__restrict__ Lin, vec2_t<T> *__restrict__ Lout,
             const vec2_t<TF> *__restrict__ LD, const vec2_t<T> *__restrict__ GX,
             vec2_t<TF> *__restrict__ Dout, T c, double *__restrict__ partials,
             const dev_status *__restrict__ status) {
    if (status->done) return;
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double fs = 0, ts = 0;
    if (s < g.V) {
        const nbr n = neighbours(g, s);
        // Eight half-steps h = 2 mu + b: b = 0 transforms the link U_mu(x)
        // with g(x+mu), b = 1 the link U_mu(x-mu) with g(x-mu).  Each needs
        // the 4 field entries of g's site (6 entries of g itself when GPRE)
        // and the LF/2 stored slots of the link; the loads of half-step h+1 are issued before
        // half-step h is computed (software pipelining), so every wave keeps
        // the next memory round trip in flight.
        constexpr int NG = GPRE ? 6 : 4;
        struct half {
            cpx<T> f[NG], u[LF / 2];
        };
        auto load_g = [&](long x, cpx<T> (&f)[NG]) {
#pragma unroll
            for (int k = 0; k < NG; ++k) {
                if constexpr (GPRE) f[k] = ld<T>(GX + (long)k * g.S + x);
                else f[k] = cvt<T>(ld<TF>(LD + (long)k * g.S + x));
            }
        };
        auto make_g = [&](const cpx<T> (&f)[NG]) {
            mat3<T> m;
            if constexpr (GPRE) {
#pragma unroll
                for (int k = 0; k < 6; ++k) m.e[k / 3][k % 3] = f[k];
                rebuild_row2(m);
            } else {
                m = gauge_from_entries<T>(f[0], f[1], f[2], f[3], c);
            }
            return m;
        };
        auto fetch = [&](int h, half &d) {
            const int mu = h >> 1;
            const long sf = (h & 1) ? n.m[mu] : n.p[mu];
            const long sl = (h & 1) ? n.m[mu] : s;
            load_g(sf, d.f);
            const vec2_t<T> *lp = Lin + (long)mu * (LF / 2) * g.S + sl;
#pragma unroll
            for (int k = 0; k < LF / 2; ++k) d.u[k] = ld<T>(lp + (long)k * g.S);
        };
        half d[2];
        cpx<T> own[NG];
        load_g(s, own);
        fetch(0, d[0]);
        const mat3<T> g0 = make_g(own);
        xacc<T> X;
        xacc_zero(X);
        T tr = 0;
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            if (h < 7) fetch(h + 1, d[(h + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            const half &cur = d[h & 1];
            const mat3<T> gn = make_g(cur.f);
            const mat3<T> u = link_from_slots<T, LF>(cur.u);
            constexpr int PR = product_rows<LF>();
            if ((h & 1) == 0) {
                const mat3<T> un = mul_abcd<PR>(g0, u, gn);  // g(x) U_mu(x) g(x+mu)^+
                if constexpr (STORE) store_link<T, LF>(Lout, g.S, h >> 1, s, un);
                tr += retrace(un);
                xacc_add(X, un, T(-1));
            } else {
                const mat3<T> umn = mul_abcd<PR>(gn, u, g0);  // g(x-mu) U_mu(x-mu) g(x)^+
                xacc_add(X, umn, T(1));
            }
        }
        cpx<T> f0, f1, f2, f3;
        ts = (double)delta_pack(X, f0, f1, f2, f3);
        fs = (double)tr;
        st_stream<TF>(Dout + s, cvt<TF>(f0));
        st_stream<TF>(Dout + g.S + s, cvt<TF>(f1));
        st_stream<TF>(Dout + 2 * g.S + s, cvt<TF>(f2));
        st_stream<TF>(Dout + 3 * g.S + s, cvt<TF>(f3));
    }
    block_sum2<SITE_BLOCK>(fs, ts, partials, blockIdx.x);
}

// ---------------------------------------------------------------------------
// the update of small lattices: a lane per half-step
// ---------------------------------------------------------------------------

// A small lattice's update is bound by the latency of one thread's chain of
// eight half-steps (and by fetching the unrolled code for them), not by memory
// or arithmetic: 9.7 us at 8^4.  Here the eight lanes of a site each form one
// link, so that all loads go out at once; a site's g is formed by all eight.
// FP64 links of 12 reals; GPRE as in k_update.  5.9 us at 8^4.
constexpr int DIR_SITES = SITE_BLOCK / 8;
inline int dir_blocks(long V) { return (int)((V + DIR_SITES - 1) / DIR_SITES); }

template <class TF, bool GPRE>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_update_dirs(geom g, const double2 *__restrict__ Lin, double2 *__restrict__ Lout,
                  const vec2_t<TF> *__restrict__ LD, const double2 *__restrict__ GX,
                  vec2_t<TF> *__restrict__ Dout, double c, double *__restrict__ partials,
                  const dev_status *__restrict__ status) {
    using T = double;
    const long s0 = (long)xcd_block(blockIdx.x, gridDim.x) * DIR_SITES + (threadIdx.x >> 3);
    const bool live = s0 < g.V;
    const long s = live ? s0 : g.V - 1;
    const int h = threadIdx.x & 7, mu = h >> 1;
    const bool in = h & 1;  // the link arriving from x - mu
    const nbr n = neighbours(g, s);
    const long sp = mu == 0 ? n.p[0] : mu == 1 ? n.p[1] : mu == 2 ? n.p[2] : n.p[3];
    const long sm = mu == 0 ? n.m[0] : mu == 1 ? n.m[1] : mu == 2 ? n.m[2] : n.m[3];
    const long q = in ? sm : sp;  // the other end of the link
    constexpr int NG = GPRE ? 6 : 4;
    cpx<T> fo[NG], fq[NG], u[6];
    auto load_g = [&](long x, cpx<T> (&f)[NG]) {
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            if constexpr (GPRE) f[k] = ld<T>(GX + (long)k * g.S + x);
            else f[k] = cvt<T>(ld<TF>(LD + (long)k * g.S + x));
        }
    };
    load_g(s, fo);
    load_g(q, fq);
    const double2 *lp = Lin + (long)mu * 6 * g.S + (in ? sm : s);
#pragma unroll
    for (int k = 0; k < 6; ++k) u[k] = ld<T>(lp + (long)k * g.S);
    if (status->done) {
        discard(fo);
        discard(fq);
        return discard(u);
    }
    // the link's ends in its own order: left at its site, right at the next
    cpx<T> fl[NG], fr[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        fl[k] = in ? fq[k] : fo[k];
        fr[k] = in ? fo[k] : fq[k];
    }
    auto make_g = [&](const cpx<T> (&f)[NG]) {
        mat3<T> m;
        if constexpr (GPRE) {
#pragma unroll
            for (int k = 0; k < 6; ++k) m.e[k / 3][k % 3] = f[k];
            rebuild_row2(m);
        } else {
            m = gauge_from_entries<T>(f[0], f[1], f[2], f[3], c);
        }
        return m;
    };
    const mat3<T> un = mul_abcd<2>(make_g(fl), link_from_slots<T, 12>(u), make_g(fr));
    if (live && !in) store_link<T, 12>(Lout, g.S, mu, s, un);
    // The sixteen reals a link adds to the divergence and to F go through LDS,
    // so that each is summed over the half-steps in the order of k_update and
    // k_div_reduce: lane h sums reals 2h and 2h + 1.
    __shared__ T X[DIR_SITES][16][9];
    T(*mine)[9] = X[threadIdx.x >> 3];
    const T sg = in ? T(1) : T(-1);
    auto put = [&](int k, cpx<T> m) {
        mine[2 * k][h] = sg * m.re;
        mine[2 * k + 1][h] = sg * m.im;
    };
    put(0, un.e[0][1]);
    put(1, un.e[1][0]);
    put(2, un.e[0][2]);
    put(3, un.e[2][0]);
    put(4, un.e[1][2]);
    put(5, un.e[2][1]);
    mine[12][h] = sg * un.e[0][0].im;
    mine[13][h] = sg * un.e[1][1].im;
    mine[14][h] = sg * un.e[2][2].im;
    mine[15][h] = in ? T(0) : retrace(un);
    __syncthreads();
    cpx<T> x = mk<T>(0, 0);
#pragma unroll
    for (int k = 0; k < 8; ++k) x = x + mk<T>(mine[2 * h][k], mine[2 * h + 1][k]);
    // lanes 2k, 2k + 1 hold the two entries of field k (lane 6 Im of the first
    // two diagonal entries, lane 7 Im of the third and the trace)
    const cpx<T> o = mk<T>(__shfl_xor(x.re, 1), __shfl_xor(x.im, 1));
    const T d0 = T(2) * x.re, d1 = T(2) * x.im, d2 = T(2) * o.re;
    const T t3 = (d0 + d1 + d2) * T(1.0 / 3.0);
    const cpx<T> f = h == 6 ? mk<T>(d0 - t3, d1 - t3) : x - conjg(o);
    if (live && (h & 1) == 0) st<TF>(Dout + (long)(h >> 1) * g.S + s, cvt<TF>(f));
    // Tr[Delta Delta^dagger], once per site
    T th = h == 6 ? f.re * f.re + f.im * f.im + (f.re + f.im) * (f.re + f.im) : T(2) * norm2(f);
    th += __shfl_xor(th, 2);
    th += __shfl_xor(th, 4);
    block_sum2<SITE_BLOCK>(live && h == 7 ? x.im : 0.0, live && h == 0 ? th : 0.0, partials,
                           blockIdx.x);
}

// ---------------------------------------------------------------------------
// FP64 sweeps that keep the input links U0 and the transformation G
// ---------------------------------------------------------------------------

// The next Delta and the partials of F and theta of the links
// U_mu(x) = G(x) U0_mu(x) G(x+mu)^dagger, which are formed and not stored: 544
// bytes per site (R U0 384, R G 96, W Delta 64) instead of the 896 of k_update
// (R links, W links, R L Delta, W Delta).  They are the links that
// k_unpack_rotated returns, rows 0,1 by products and row 2 completed from them,
// also where U0 is in SU(3) only to the precision it was stored in.  With q(A)
// for rows 0,1 of A and their completion, and as completing commutes with an
// SU(3) factor on the right,
//   sum_mu U_mu(x-mu)^dagger = G(x) sum_mu q(G(x-mu) U0_mu(x-mu))^dagger
// while of the links leaving x, with p = q(U0 G(x+mu)^dagger), rows 0,1 are
// those of G(x) p and row 2 is that of G(x) p', p' the conjugate cofactors of p
// (p itself in SU(3); always p's third row).  So the sum over mu of U_mu(x) +
// U_mu(x-mu)^dagger is M with rows 0,1 of G(x) K(x) and row 2 of G(x) K'(x),
// K and K' the sums of the q^dagger with the p and with the p', X - X^dagger =
// M^dagger - M, and the eight links need nine matrix products instead of
// sixteen; sum_mu Re Tr U_mu over the lattice is half that of M.  Row 2 from K
// as well (the links formed in SU(3) throughout) makes a solve of links rounded
// to FP32 stop at theta = 7e-16 of M where the returned links have 2e-15, and
// saves 1% (27^4 85.7 against 86.1 us, 24^4 43.5 against 44.5).
// With K alone at 32^4 146 us against 195 for k_update (event timing; 725 MB of
// measured traffic against 1060): the time of its reads, as a kernel that only
// streams U0 and G and writes Delta takes 122 us, and one whose eight
// neighbours are its own site 142.  222 VGPRs, two waves per SIMD: with three
// (168 VGPRs) 152 us, with four and no load ahead 169, as more blocks in
// flight find fewer neighbour lines in L2.  Marking the loads of U0 as
// streaming costs the L2 reuse of U0(x-mu): 171 us.  Taking the arriving links
// before the leaving ones costs reuse too (24^4 52, 27^4 92 us).
template <class TF>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_update_u0(geom g, const double2 *__restrict__ U0, const double2 *__restrict__ G,
                vec2_t<TF> *__restrict__ Dout, double *__restrict__ partials,
                const dev_status *__restrict__ status) {
    using T = double;
    if (status->done) return;
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double fs = 0, ts = 0;
    if (s < g.V) {
        const nbr n = neighbours(g, s);
        struct half {
            cpx<T> f[6], u[6];
        };
        // half-steps h = 2 mu + b as in k_update: b = 0 the link leaving x, b = 1
        // the one arriving from x - mu; one ahead in flight
        auto fetch = [&](int h, half &d) {
            const int mu = h >> 1;
            const long sf = (h & 1) ? n.m[mu] : n.p[mu];
            const long sl = (h & 1) ? n.m[mu] : s;
#pragma unroll
            for (int k = 0; k < 6; ++k) d.f[k] = ld<T>(G + (long)k * g.S + sf);
            const double2 *lp = U0 + (long)mu * 6 * g.S + sl;
#pragma unroll
            for (int k = 0; k < 6; ++k) d.u[k] = ld<T>(lp + (long)k * g.S);
        };
        auto rows01 = [](const cpx<T> (&f)[6]) {
            mat3<T> m;
#pragma unroll
            for (int k = 0; k < 6; ++k) m.e[k / 3][k % 3] = f[k];
            return m;
        };
        half d[2];
        fetch(0, d[0]);
        mat3<T> K;
        cpx<T> C[2][3];  // rows 0,1 of K' (row 2 is that of K)
#pragma unroll
        for (int k = 0; k < 9; ++k) K.e[k / 3][k % 3] = mk<T>(0, 0);
#pragma unroll
        for (int k = 0; k < 6; ++k) C[k / 3][k % 3] = mk<T>(0, 0);
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            if (h < 7) fetch(h + 1, d[(h + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            const half &cur = d[h & 1];
            mat3<T> gn = rows01(cur.f), u = rows01(cur.u), p;
            if ((h & 1) == 0) {
                rebuild_row2(gn);  // rows 0,1 of U0 G^dagger need rows 0,1 of U0
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        cpx<T> a = cmulc(u.e[i][0], gn.e[j][0]);
                        a = cmacc(a, u.e[i][1], gn.e[j][1]);
                        p.e[i][j] = cmacc(a, u.e[i][2], gn.e[j][2]);
                    }
                rebuild_row2(p);
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    K.e[k / 3][k % 3] = K.e[k / 3][k % 3] + p.e[k / 3][k % 3];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const int r = i + 1, t = (i + 2) % 3, a = (j + 1) % 3, b = (j + 2) % 3;
                        const cpx<T> m = cmul(p.e[r][a], p.e[t][b]);
                        C[i][j] = C[i][j] + conjg(cmsub(m, p.e[r][b], p.e[t][a]));
                    }
            } else {
                rebuild_row2(u);  // rows 0,1 of G U0 need rows 0,1 of G
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        cpx<T> a = cmul(gn.e[i][0], u.e[0][j]);
                        a = cmac(a, gn.e[i][1], u.e[1][j]);
                        p.e[i][j] = cmac(a, gn.e[i][2], u.e[2][j]);
                    }
                rebuild_row2(p);
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    K.e[k / 3][k % 3] = K.e[k / 3][k % 3] + conjg(p.e[k % 3][k / 3]);
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    C[k / 3][k % 3] = C[k / 3][k % 3] + conjg(p.e[k % 3][k / 3]);
            }
        }
        mat3<T> g0;
#pragma unroll
        for (int k = 0; k < 6; ++k) g0.e[k / 3][k % 3] = ld<T>(G + (long)k * g.S + s);
        rebuild_row2(g0);
        mat3<T> M;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                cpx<T> a = cmul(g0.e[i][0], i < 2 ? K.e[0][j] : C[0][j]);
                a = cmac(a, g0.e[i][1], i < 2 ? K.e[1][j] : C[1][j]);
                M.e[i][j] = cmac(a, g0.e[i][2], K.e[2][j]);
            }
        xacc<T> X;
        xacc_zero(X);
        xacc_add(X, M, T(-1));
        fs = 0.5 * retrace(M);
        cpx<T> f0, f1, f2, f3;
        ts = delta_pack(X, f0, f1, f2, f3);
        st_stream<TF>(Dout + s, cvt<TF>(f0));
        st_stream<TF>(Dout + g.S + s, cvt<TF>(f1));
        st_stream<TF>(Dout + 2 * g.S + s, cvt<TF>(f2));
        st_stream<TF>(Dout + 3 * g.S + s, cvt<TF>(f3));
    }
    block_sum2<SITE_BLOCK>(fs, ts, partials, blockIdx.x);
}

// The caller's links G(x) U0_mu(x) G(x+mu)^dagger at the end of such a phase.
// A wave's 64 sites are consecutive (block_site), so each wave stages its 64
// links of one direction in LDS and writes them as one contiguous run.
__global__ void __launch_bounds__(SITE_BLOCK)
    k_unpack_rotated(geom g, const double2 *__restrict__ U0, const double2 *__restrict__ G,
                     double2 *__restrict__ U) {
    __shared__ double2 buf[SITE_BLOCK * 9];
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    const int lane = threadIdx.x & 63;
    double2 *mine = buf + (threadIdx.x - lane) * 9;
    const long s0 = s - lane;  // first site of the wave
    const int cnt = (int)(g.V - s0 < 64 ? (g.V > s0 ? g.V - s0 : 0) : 64) * 9;
    const bool live = s < g.V;
    nbr n{};
    mat3<double> g0;
    auto load_G = [&](long q) {
        mat3<double> m;
#pragma unroll
        for (int k = 0; k < 6; ++k) m.e[k / 3][k % 3] = ld<double>(G + (long)k * g.S + q);
        rebuild_row2(m);
        return m;
    };
    if (live) {
        n = neighbours(g, s);
        g0 = load_G(s);
    }
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        if (live) {
            const mat3<double> r =
                mul_abcd<2>(g0, load_link<double, 12>(U0, g.S, mu, s), load_G(n.p[mu]));
#pragma unroll
            for (int k = 0; k < 9; ++k)
                mine[lane * 9 + k] = make_double2(r.e[k / 3][k % 3].re, r.e[k / 3][k % 3].im);
        }
        __syncthreads();
        double2 *u = U + ((long)mu * g.V + s0) * 9;
        for (int e = lane; e < cnt; e += 64) u[e] = mine[e];
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// sweeps that keep U0 and G with the links shared through LDS
// ---------------------------------------------------------------------------

// Every link U_mu(x) enters two divergences: with sign - at x and with sign +
// at x + mu, so k_update forms each link twice.  The divergence is linear in
// the links through P(M): the off-diagonal differences M_ij - conj(M_ji)
// (i < j) and the traceless part of 2 Im M_ii, 8 reals, in the order of the 4
// Fourier-field entries.  This kernel forms the 4 links leaving each site,
// keeps their P in LDS and takes the links arriving from x - mu from LDS when
// x - mu is in the block, forming them again otherwise.  A block holds
// UPDS_XY consecutive xy-sites at UPDS_T consecutive t and one z: the x
// neighbour is in the block whenever UPDS_XY is a multiple of Lx, the y
// neighbour except in the block's first xy-row, the t neighbour except at
// its first t, the z neighbour never.  Arithmetic as in k_update; the
// per-link projections change the rounding order of the sums, not the
// quantities.  Partial sums go out per group of SITE_BLOCK threads, so the
// finalize reads the same number of partials as after k_update.
// Blocks of 128 xy-sites x 4 t (512 threads, 48 KB of LDS) let two blocks
// share a compute unit (their registers allow no third), so that one block's
// loads overlap the other's arithmetic: with the z links' P in LDS as well (64
// KB) 73 against 82 us at 32^4 and 797 against 828 us at 48^3 x 96 for one block
// of 256 x 4 (or 256 x 2: 74 / 848 us; 128 x 2: 73 / 855 us).
// Lattices with less than one such block per compute unit take blocks of 64 x 4.
constexpr int UPDS_T = 4;
constexpr long UPDS_SPLIT_SITES = 131072;
template <class T, int XY> constexpr size_t upds_lds() { return (size_t)8 * 3 * XY * UPDS_T * sizeof(T); }
static_assert(upds_lds<float, 128>() == 48 * 1024 && upds_lds<double, 64>() == 48 * 1024,
              "the update is launched without raising the LDS limit of 64 KB");

// FP32: the loads of U0's x, y and t links (each read once by its own block)
// are streaming where the sweep's data do not fit the 256 MB last-level cache
// but all besides U0 (G twice, the field twice: 160 bytes per site) do: what
// the next kernels read then stays there (32^4: sweep 154 -> 147 us, the
// transforms 73 -> 68; 48^3 x 96, where nothing fits, 1681 -> 1715).
inline bool upds_stream(const geom &g) {
    const double mall = 256.0 * 1024 * 1024;
    return 368.0 * g.V > mall && 160.0 * g.V < mall;
}

// FP64 (sweeps that keep U0 and G): blocks of 64 x 4, two per compute unit, two
// waves per SIMD, where k_update_u0's neighbour reads leave L2: 32^4 147 -> 136
// us, 24^3 x 48 98 -> 94, 48^3 x 96 1531 -> 1512, but 16^2 x 32^2 32.5 -> 33.4
// and 24^4 44.5 -> 47.3.  Streaming loads do not help here (136 -> 140).
inline bool update_shared64_ok(const geom &g) {
    return g.keeps_u0() && g.V >= 524288 && (long)g.Lx * g.Ly % 64 == 0 && g.Lt % UPDS_T == 0;
}

inline bool update_shared_ok(const geom &g) {
    const long Lxy = (long)g.Lx * g.Ly;
    return g.nc == 3 && g.lf == 12 && Lxy % 128 == 0 && g.Lt % UPDS_T == 0;
}

// block sum of two doubles per group of NG threads into partials[2 * (slot0 + group) + {0,1}]
template <int NT, int NG>
__device__ __forceinline__ void group_sum2(double a, double b, double *partials, int slot0) {
    static_assert(NT % NG == 0 && NG % 64 == 0, "wave64 groups");
    __shared__ double sa[NT / 64], sb[NT / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off);
        b += __shfl_xor(b, off);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sa[w] = a;
        sb[w] = b;
    }
    __syncthreads();
    if (threadIdx.x % NG == 0) {
        const int w0 = threadIdx.x >> 6;
        double A = 0, B = 0;
#pragma unroll
        for (int i = 0; i < NG / 64; ++i) {
            A += sa[w0 + i];
            B += sb[w0 + i];
        }
        const int slot = slot0 + threadIdx.x / NG;
        partials[2 * slot] = A;
        partials[2 * slot + 1] = B;
    }
}

// FP32: four waves per SIMD, two blocks per compute unit (at most 128 VGPRs);
// FP64: two and 256
__device__ constexpr int mu_slot(int mu) { return mu == 3 ? 2 : mu; }

template <class T, class TF, int UPDS_XY, bool STREAM>
__global__ void __launch_bounds__(UPDS_XY * UPDS_T)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
    k_update_shared(geom g, const vec2_t<T> *__restrict__ Lin, const vec2_t<T> *__restrict__ GX,
                    vec2_t<TF> *__restrict__ Dout, double *__restrict__ partials,
                    const dev_status *__restrict__ status) {
    constexpr int UPDS_THREADS = UPDS_XY * UPDS_T;
    if (status->done) return;
    extern __shared__ unsigned char smem_raw[];
    T *P = reinterpret_cast<T *>(smem_raw);  // P[(k * 3 + mu_slot) * UPDS_THREADS + i], x, y, t
    // block -> (z fastest, then the xy group, then the t group); XCDs walk
    // contiguous ranges
    const int B = xcd_block(blockIdx.x, gridDim.x);
    const unsigned Lxy = (unsigned)g.Lx * (unsigned)g.Ly, ngxy = Lxy / UPDS_XY;
    const unsigned z = (unsigned)B % (unsigned)g.Lz, r = (unsigned)B / (unsigned)g.Lz;
    const unsigned xy0 = (r % ngxy) * UPDS_XY, t0 = (r / ngxy) * UPDS_T;
    const int i = threadIdx.x;  // local index: (t - t0) * UPDS_XY + (xy - xy0)
    const unsigned xy = xy0 + (unsigned)i % UPDS_XY, t = t0 + (unsigned)i / UPDS_XY;
    const unsigned s = xy + Lxy * (z + (unsigned)g.Lz * t);
    const unsigned x = xy % (unsigned)g.Lx, y = (xy / (unsigned)g.Lx) % (unsigned)g.Ly;
    const unsigned Lx = g.Lx, Ly = g.Ly, Lz = g.Lz, Lt = g.Lt, sz = Lxy, st = Lxy * Lz;
    // neighbour s + mu (fwd) or s - mu, periodic, in 32-bit arithmetic (V < 2^31)
    auto nb = [&](int mu, bool fwd) -> unsigned {
        if (mu == 0) return fwd ? (x == Lx - 1 ? s - (Lx - 1) : s + 1) : (x == 0 ? s + (Lx - 1) : s - 1);
        if (mu == 1)
            return fwd ? (y == Ly - 1 ? s - (Ly - 1) * Lx : s + Lx) : (y == 0 ? s + (Ly - 1) * Lx : s - Lx);
        if (mu == 2)
            return fwd ? (z == Lz - 1 ? s - (Lz - 1) * sz : s + sz) : (z == 0 ? s + (Lz - 1) * sz : s - sz);
        return fwd ? (t == Lt - 1 ? s - (Lt - 1) * st : s + st) : (t == 0 ? s + (Lt - 1) * st : s - st);
    };
    const long S = g.S;
    auto load_g = [&](unsigned q, cpx<T> (&f)[6]) {
#pragma unroll
        for (int k = 0; k < 6; ++k) f[k] = ld<T>(GX + (long)k * S + q);
    };
    auto make_g = [&](const cpx<T> (&f)[6]) {
        mat3<T> m;
#pragma unroll
        for (int k = 0; k < 6; ++k) m.e[k / 3][k % 3] = f[k];
        rebuild_row2(m);
        return m;
    };
    struct half {
        cpx<T> f[6], u[6];
    };
    // h = 2 mu + b as in k_update: b = 0 the link leaving x, b = 1 the one arriving from x - mu
    auto fetch = [&](int h, half &d, bool halo = false) {
        const int mu = h >> 1;
        const unsigned sf = nb(mu, (h & 1) == 0);
        const unsigned sl = (h & 1) ? sf : s;
        load_g(sf, d.f);
        const vec2_t<T> *lp = Lin + (long)mu * 6 * S + sl;
        // the z links are read by two blocks and come from L2 the second time
        const bool stream = STREAM && mu != 2 && (halo || (h & 1) == 0);
#pragma unroll
        for (int k = 0; k < 6; ++k)
            d.u[k] = stream ? ld_stream<T>(lp + (long)k * S) : ld<T>(lp + (long)k * S);
    };
    cpx<T> own[6];
    load_g(s, own);
    half d[2];
    fetch(0, d[0]);
    const mat3<T> g0 = make_g(own);
    T X[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) X[k] = T(0);
    T tr = 0;
    // links leaving x: U_mu(x) = g(x) U0_mu(x) g(x+mu)^+; the z link arriving
    // from x - z (never in the block) is fetched during the last of them
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        fetch(mu < 3 ? 2 * (mu + 1) : 5, d[(mu + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        const half &cur = d[mu & 1];
        const mat3<T> un = mul_abcd<2>(g0, link_from_slots<T, 12>(cur.u), make_g(cur.f));
        tr += retrace(un);
        T pm[8];
        proj_of(pm, un);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (mu != 2) P[(k * 3 + mu_slot(mu)) * UPDS_THREADS + i] = pm[k];
            X[k] -= pm[k];
        }
    }
    // the z link arriving from x - z: g(x-z) U0_z(x-z) g(x)^+
    {
        const half &cur = d[0];
        const mat3<T> umn = mul_abcd<2>(make_g(cur.f), link_from_slots<T, 12>(cur.u), g0);
        proj_add(X, umn, T(1));
    }
    __syncthreads();
    // x, y, t links arriving from x - mu: from LDS inside the block
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        if (mu == 2) continue;
        unsigned txy = xy, tt = t;
        if (mu == 0) txy = x == 0 ? xy + Lx - 1 : xy - 1;
        if (mu == 1) txy = y == 0 ? xy + (Ly - 1) * Lx : xy - Lx;
        if (mu == 3) tt = t == 0 ? Lt - 1 : t - 1;
        const unsigned lx = txy - xy0, lt = tt - t0;
        if (lx < (unsigned)UPDS_XY && lt < (unsigned)UPDS_T) {
            const int j = (int)(lt * UPDS_XY + lx);
#pragma unroll
            for (int k = 0; k < 8; ++k) X[k] += P[(k * 3 + mu_slot(mu)) * UPDS_THREADS + j];
        } else {
            half e;
            fetch(2 * mu + 1, e, true);
            const mat3<T> umn = mul_abcd<2>(make_g(e.f), link_from_slots<T, 12>(e.u), g0);
            proj_add(X, umn, T(1));
        }
    }
    const cpx<T> f0 = mk<T>(X[0], X[1]), f1 = mk<T>(X[2], X[3]), f2 = mk<T>(X[4], X[5]),
                 f3 = mk<T>(X[6], X[7]);
    const T da = X[6], db = X[7];
    const T th = T(2) * (norm2(f0) + norm2(f1) + norm2(f2)) + da * da + db * db + (da + db) * (da + db);
    st_stream<TF>(Dout + s, cvt<TF>(f0));
    st_stream<TF>(Dout + S + s, cvt<TF>(f1));
    st_stream<TF>(Dout + 2 * S + s, cvt<TF>(f2));
    st_stream<TF>(Dout + 3 * S + s, cvt<TF>(f3));
    group_sum2<UPDS_THREADS, SITE_BLOCK>((double)tr, (double)th, partials,
                                         blockIdx.x * (UPDS_THREADS / SITE_BLOCK));
}

// reorder 4 fields between natural index order and transform-position order
__global__ void k_reorder(geom g, const double2 *__restrict__ in, long si, double2 *__restrict__ out,
                          long so, int to_natural) {
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.V) return;
    long r = s;
    const int a0 = (int)(r % g.Lx); r /= g.Lx;
    const int a1 = (int)(r % g.Ly); r /= g.Ly;
    const int a2 = (int)(r % g.Lz);
    const int a3 = (int)(r / g.Lz);
    // s is a position index; its natural (frequency) index:
    const int f0 = fft_freq_of_pos(g.Lx, a0), f1 = fft_freq_of_pos(g.Ly, a1),
              f2 = fft_freq_of_pos(g.Lz, a2), f3 = fft_freq_of_pos(g.Lt, a3);
    const long sn = f0 + (long)g.Lx * (f1 + (long)g.Ly * (f2 + (long)g.Lz * f3));
    for (int f = 0; f < 4; ++f) {
        if (to_natural) out[f * so + sn] = in[f * si + s];
        else out[f * so + s] = in[f * si + sn];
    }
}

__global__ void __launch_bounds__(FIN_BLOCK)
    k_finalize(const double *__restrict__ partials, int nparts, dev_status *__restrict__ status,
               fin_params fp) {
    dev_status st = *status;
    if (!st.done) {
        double A, B;
        if (nparts <= FOLD_MAX_PARTS) wave_sum(partials, nparts, A, B);  // launched with one wave
        else fixed_order_sum<FIN_BLOCK>(partials, nparts, A, B);
        st = next_state(A, B, st, fp, threadIdx.x == 0);
        if (threadIdx.x == 0) *status = st;
    }
    // straight into pinned host memory: a copy of its own would be another
    // launch per batch of sweeps
    if (threadIdx.x == 0 && fp.host) {
        *fp.host = st;
        __threadfence_system();
    }
}

__global__ void k_status_reset(dev_status *status, int hist_base) {
    dev_status st;
    st.F = 0;
    st.theta = 0;
    st.theta_prev = 0;
    st.theta_min = 0;
    st.n = 0;
    st.done = 0;
    st.code = ST_RUNNING;
    st.rises = 0;
    st.hist_base = hist_base;
    st.since_min = 0;
    *status = st;
}

__global__ void __launch_bounds__(FIN_BLOCK)
    k_measure_finalize(const double *__restrict__ partials, int nparts, double *out2,
                       double normF, double normT) {
    double A, B;
    fixed_order_sum<FIN_BLOCK>(partials, nparts, A, B);
    if (threadIdx.x == 0) {
        out2[0] = A * normF;
        out2[1] = B * normT;
    }
}

__global__ void __launch_bounds__(FIN_BLOCK)
    k_reduce_only(const double *__restrict__ partials, int nparts, double *out2) {
    double A, B;
    fixed_order_sum<FIN_BLOCK>(partials, nparts, A, B);
    if (threadIdx.x == 0) {
        out2[0] = A;
        out2[1] = B;
    }
}

// ---------------------------------------------------------------------------
// mixed precision: accumulated transformation and the hand-over to FP64
// ---------------------------------------------------------------------------

__global__ void k_g_identity(float2 *__restrict__ G, long V, long S) {
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
#pragma unroll
    for (int k = 0; k < 6; ++k) G[(long)k * S + s] = make_float2(k == 0 || k == 4 ? 1.f : 0.f, 0.f);
}

__device__ __forceinline__ mat3<double> load_G_fp64(const float2 *__restrict__ G, long S, long s) {
    mat3<double> m;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        float2 v = G[(long)k * S + s];
        m.e[k / 3][k % 3] = mk<double>(v.x, v.y);
    }
    reunitarise(m);
    return m;
}

// U_mu(x) = G(x) U0_mu(x) G(x+mu)^dagger in FP64, G reunitarised in FP64
template <int LF>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_switch(geom g, const float2 *__restrict__ G, const double2 *__restrict__ U0,
             double2 *__restrict__ L) {
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.V) return;
    const nbr n = neighbours(g, s);
    const mat3<double> g0 = load_G_fp64(G, g.S, s);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        const mat3<double> gp = load_G_fp64(G, g.S, n.p[mu]);
        const mat3<double> u = aos_link<double, LF>(U0 + ((long)mu * g.V + s) * 9);
        store_link<double, LF>(L, g.S, mu, s, mul_abcd<product_rows<LF>()>(g0, u, gp));
    }
}

// The hand-over fused with the first FP64 divergence: the links of x as in
// k_switch (stored), the links U_mu(x-mu) formed again from G(x-mu), U0 and
// G(x) exactly as their own site forms them, then Delta(x) and the block
// partials of F and theta, as k_div_reduce would compute them from the stored
// links (the same values in the same order).
template <int LF, class TF>
__global__ void __launch_bounds__(SITE_BLOCK)
    k_switch_div(geom g, const float2 *__restrict__ G, const double2 *__restrict__ U0,
                 double2 *__restrict__ L, vec2_t<TF> *__restrict__ D, double *__restrict__ partials) {
    const long s = block_site(g, blockIdx.x, gridDim.x, threadIdx.x);
    double fs = 0, ts = 0;
    if (s < g.V) {
        const nbr n = neighbours(g, s);
        const mat3<double> g0 = load_G_fp64(G, g.S, s);
        xacc<double> X;
        xacc_zero(X);
        double tr = 0;
        auto aos = [&](int mu, long x) { return aos_link<double, LF>(U0 + ((long)mu * g.V + x) * 9); };
        constexpr int PR = product_rows<LF>();
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const mat3<double> un = mul_abcd<PR>(g0, aos(mu, s), load_G_fp64(G, g.S, n.p[mu]));
            store_link<double, LF>(L, g.S, mu, s, un);
            const mat3<double> u = as_stored<double, LF>(un);  // as loaded back
            tr += retrace(u);
            xacc_add(X, u, -1.0);
            const mat3<double> um =
                as_stored<double, LF>(mul_abcd<PR>(load_G_fp64(G, g.S, n.m[mu]), aos(mu, n.m[mu]), g0));
            xacc_add(X, um, 1.0);
        }
        cpx<double> f0, f1, f2, f3;
        ts = delta_pack(X, f0, f1, f2, f3);
        fs = tr;
        st<TF>(D + s, cvt<TF>(f0));
        st<TF>(D + g.S + s, cvt<TF>(f1));
        st<TF>(D + 2 * g.S + s, cvt<TF>(f2));
        st<TF>(D + 3 * g.S + s, cvt<TF>(f3));
    }
    block_sum2<SITE_BLOCK>(fs, ts, partials, blockIdx.x);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline unsigned nblk(long n, int b) { return (unsigned)((n + b - 1) / b); }

static void finalize(const double *partials, int nparts, dev_status *status, const fin_params &fp,
                     hipStream_t st) {
    k_finalize<<<1, nparts <= FOLD_MAX_PARTS ? 64 : FIN_BLOCK, 0, st>>>(partials, nparts, status, fp);
}

template <class T>
hipError_t launch_pack_links(const double *Uaos, void *L, const geom &g, hipStream_t st) {
    if (g.nc == 2) return launch_pack_su2<T>(Uaos, L, g, st);
    auto U = reinterpret_cast<const double2 *>(Uaos);
    auto Lp = static_cast<vec2_t<T> *>(L);
    const long V = g.V, S = g.S;
    if (g.lf == 18) k_pack_links<T, 18><<<nblk(4 * V, 256), 256, 0, st>>>(U, Lp, V, S);
    else if (g.lf == 8) k_pack_links<T, 8><<<nblk(4 * V, 256), 256, 0, st>>>(U, Lp, V, S);
    else k_pack_links<T, 12><<<nblk(4 * V, 256), 256, 0, st>>>(U, Lp, V, S);
    return hipGetLastError();
}
template hipError_t launch_pack_links<double>(const double *, void *, const geom &, hipStream_t);
template hipError_t launch_pack_links<float>(const double *, void *, const geom &, hipStream_t);

hipError_t launch_unpack_links(const void *L64, double *Uaos, const geom &g, hipStream_t st) {
    if (g.nc == 2) return launch_unpack_su2(L64, Uaos, g, st);
    auto Lp = static_cast<const double2 *>(L64);
    auto U = reinterpret_cast<double2 *>(Uaos);
    const long V = g.V, S = g.S;
    if (g.lf == 18) k_unpack_links<18><<<nblk(4 * V, 256), 256, 0, st>>>(Lp, U, V, S);
    else if (g.lf == 8) k_unpack_links<8><<<nblk(4 * V, 256), 256, 0, st>>>(Lp, U, V, S);
    else k_unpack_links<12><<<nblk(4 * V, 256), 256, 0, st>>>(Lp, U, V, S);
    return hipGetLastError();
}

// g(x) = exp((alpha/2) L Delta(x)) exactly, once per site, rows 0,1 into GX
// (the update then reads it at x and its neighbours instead of evaluating the
// series nine times per site).
template <class T, class TF>
__global__ void __launch_bounds__(256)
    k_gauge_exp(geom g, const vec2_t<TF> *__restrict__ LD, vec2_t<T> *__restrict__ GX, T c,
                const dev_status *__restrict__ status) {
    if (status->done) return;
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.V) return;
    const mat3<T> m = gauge_exp_from_entries<T>(
        cvt<T>(ld<TF>(LD + s)), cvt<T>(ld<TF>(LD + g.S + s)), cvt<T>(ld<TF>(LD + 2 * g.S + s)),
        cvt<T>(ld<TF>(LD + 3 * g.S + s)), c);
#pragma unroll
    for (int k = 0; k < 6; ++k) st<T>(GX + (long)k * g.S + s, m.e[k / 3][k % 3]);
}

// Sweeps that keep U0 and G: G(x) <- g(x) G(x), rows 0,1 kept (12 reals),
// from Gold into Gnew (the update then forms G(x) U0 G(x+mu)^dagger at x and
// its neighbours from Gnew; the old G stays readable for those neighbours).
// g and the product are formed and reunitarised in FP64 (accumulate_G).
template <bool EXACT, class TF, class TG>
__global__ void __launch_bounds__(256)
    k_gauge_acc(geom g, const vec2_t<TF> *__restrict__ LD, const vec2_t<TG> *__restrict__ Gold,
                vec2_t<TG> *__restrict__ Gnew, double c, const dev_status *__restrict__ status) {
    if (status->done) return;
    const long s = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.V) return;
    accumulate_G<EXACT, TF, TG>(ld<TF>(LD + s), ld<TF>(LD + g.S + s), ld<TF>(LD + 2 * g.S + s),
                                ld<TF>(LD + 3 * g.S + s), c, Gold, Gnew, g.S, s);
}

// The Fourier field is FP32 for FP32 sweeps and, when g.ff32 is set, for FP64
// sweeps too; f(tag) runs the body with the field's real type.
template <class T, class Body> hipError_t with_field_type(const geom &g, Body f) {
    if constexpr (std::is_same<T, double>::value) {
        if (g.ff32) return f(float{});
        return f(double{});
    } else {
        return f(float{});
    }
}

template <class T>
hipError_t launch_div_reduce(const geom &g, const void *L, void *D, double *partials,
                             dev_status *status, const fin_params &fp, hipStream_t st) {
    const hipError_t e = with_field_type<T>(g, [&](auto tf) -> hipError_t {
        using TF = decltype(tf);
        auto Lp = static_cast<const vec2_t<T> *>(L);
        auto Dp = static_cast<vec2_t<TF> *>(D);
        if (g.nc == 2) return launch_div_reduce_su2<T, TF>(g, L, D, partials, status, st);
        if (g.lf == 18)
            k_div_reduce<T, TF, 18>
                <<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Lp, Dp, partials, status);
        else if (g.lf == 8)
            k_div_reduce<T, TF, 8>
                <<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Lp, Dp, partials, status);
        else
            k_div_reduce<T, TF, 12>
                <<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Lp, Dp, partials, status);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    if (fp.enabled) finalize(partials, site_blocks(g.V), status, fp, st);
    return hipGetLastError();
}
template hipError_t launch_div_reduce<double>(const geom &, const void *, void *, double *,
                                              dev_status *, const fin_params &, hipStream_t);
template hipError_t launch_div_reduce<float>(const geom &, const void *, void *, double *,
                                             dev_status *, const fin_params &, hipStream_t);

template <class T>
hipError_t launch_update(const geom &g, const void *Lin, void *Lout, const void *LD, void *Dout,
                         void *G, T c, bool exact, void *GX, double *partials, dev_status *status,
                         const fin_params &fp, hipStream_t st) {
    // G (the accumulated transformation) exists only in the FP32 phase
    constexpr bool ACC = std::is_same<T, float>::value;
    if ((G != nullptr) != ACC) return hipErrorInvalidValue;
    const hipError_t e = with_field_type<T>(g, [&](auto tf) -> hipError_t {
        using TF = decltype(tf);
        if (g.nc == 2)
            return launch_update_su2<T, TF>(g, Lin, Lout, LD, Dout, G, c, exact, partials, status,
                                            st);
        auto LDp = static_cast<const vec2_t<TF> *>(LD);
        if (ACC || exact) {
            if (!GX) return hipErrorInvalidValue;
            // FP32: GX already holds g G (launch_fft_xy_inv_acc / launch_gauge_acc)
            if constexpr (!ACC)
                k_gauge_exp<T, TF><<<nblk(g.V, 256), 256, 0, st>>>(
                    g, LDp, static_cast<vec2_t<T> *>(GX), c, status);
        }
        auto go = [&](auto kernel) {
            kernel<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(
                g, static_cast<const vec2_t<T> *>(Lin), static_cast<vec2_t<T> *>(Lout), LDp,
                static_cast<const vec2_t<T> *>(GX), static_cast<vec2_t<TF> *>(Dout), c, partials,
                status);
        };
        if constexpr (ACC) {
            // links G U0 G^dagger from the constant copy U0 (Lin), not stored
            if (update_shared_ok(g)) {
                auto shared = [&](auto xy, auto stream) {
                    constexpr int XY = decltype(xy)::value;
                    k_update_shared<float, float, XY, decltype(stream)::value>
                        <<<(unsigned)(g.V / (XY * UPDS_T)), XY * UPDS_T, upds_lds<float, XY>(), st>>>(
                            g, static_cast<const float2 *>(Lin), static_cast<const float2 *>(GX),
                            static_cast<float2 *>(Dout), partials, status);
                };
                using N64 = std::integral_constant<int, 64>;
                using N128 = std::integral_constant<int, 128>;
                if (g.V < UPDS_SPLIT_SITES) shared(N64{}, std::false_type{});
                else if (upds_stream(g)) shared(N128{}, std::true_type{});
                else shared(N128{}, std::false_type{});
                return hipGetLastError();
            }
            if (g.lf == 18) go(k_update<T, TF, true, 18, false>);
            else if (g.lf == 8) go(k_update<T, TF, true, 8, false>);
            else go(k_update<T, TF, true, 12, false>);
        } else if (g.lf == 18) {
            if (exact) go(k_update<T, TF, true, 18, true>);
            else go(k_update<T, TF, false, 18, true>);
        } else if (g.lf == 8) {
            if (exact) go(k_update<T, TF, true, 8, true>);
            else go(k_update<T, TF, false, 8, true>);
        } else {
            if (exact) go(k_update<T, TF, true, 12, true>);
            else go(k_update<T, TF, false, 12, true>);
        }
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    if (fp.enabled) finalize(partials, site_blocks(g.V), status, fp, st);
    return hipGetLastError();
}
template <class TF, class TG>
hipError_t launch_gauge_acc(const geom &g, const void *LD, const void *Gold, void *Gnew, double c,
                            bool exact, const dev_status *status, hipStream_t st) {
    if (g.nc != 3) return hipErrorInvalidValue;
    auto LDp = static_cast<const vec2_t<TF> *>(LD);
    auto Go = static_cast<const vec2_t<TG> *>(Gold);
    auto Gn = static_cast<vec2_t<TG> *>(Gnew);
    if (exact)
        k_gauge_acc<true, TF, TG><<<nblk(g.V, 256), 256, 0, st>>>(g, LDp, Go, Gn, c, status);
    else
        k_gauge_acc<false, TF, TG><<<nblk(g.V, 256), 256, 0, st>>>(g, LDp, Go, Gn, c, status);
    return hipGetLastError();
}
template hipError_t launch_gauge_acc<float, float>(const geom &, const void *, const void *, void *,
                                                   double, bool, const dev_status *, hipStream_t);
template hipError_t launch_gauge_acc<float, double>(const geom &, const void *, const void *,
                                                    void *, double, bool, const dev_status *,
                                                    hipStream_t);
template hipError_t launch_gauge_acc<double, double>(const geom &, const void *, const void *,
                                                     void *, double, bool, const dev_status *,
                                                     hipStream_t);

int update_dirs_parts(const geom &g) { return dir_blocks(g.V); }

hipError_t launch_update_dirs(const geom &g, const void *Lin, void *Lout, const void *LD,
                              void *Dout, double c, bool exact, void *GX, double *partials,
                              dev_status *status, const fin_params &fp, hipStream_t st) {
    if (g.nc != 3 || g.lf != 12) return hipErrorInvalidValue;
    const int nb = dir_blocks(g.V);
    auto Li = static_cast<const double2 *>(Lin);
    auto Lo = static_cast<double2 *>(Lout);
    auto G = static_cast<double2 *>(GX);
    auto go = [&](auto tf) {
        using TF = decltype(tf);
        auto LDp = static_cast<const vec2_t<TF> *>(LD);
        auto Dp = static_cast<vec2_t<TF> *>(Dout);
        if (exact) {
            k_gauge_exp<double, TF><<<nblk(g.V, 256), 256, 0, st>>>(g, LDp, G, c, status);
            k_update_dirs<TF, true><<<nb, SITE_BLOCK, 0, st>>>(g, Li, Lo, LDp, G, Dp, c, partials, status);
        } else {
            k_update_dirs<TF, false><<<nb, SITE_BLOCK, 0, st>>>(g, Li, Lo, LDp, G, Dp, c, partials, status);
        }
    };
    if (exact && !GX) return hipErrorInvalidValue;
    if (g.ff32) go(float{});
    else go(double{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !fp.enabled) return e;
    finalize(partials, nb, status, fp, st);
    return hipGetLastError();
}

hipError_t launch_update_u0(const geom &g, const void *U0, const void *G, void *Dout,
                            double *partials, dev_status *status, const fin_params &fp,
                            hipStream_t st) {
    if (!g.keeps_u0()) return hipErrorInvalidValue;
    auto go = [&](auto kernel, auto *D) {
        kernel<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, static_cast<const double2 *>(U0),
                                                        static_cast<const double2 *>(G), D,
                                                        partials, status);
    };
    auto shared = [&](auto *D) {
        using TF = decltype(D->x);
        k_update_shared<double, TF, 64, false>
            <<<(unsigned)(g.V / SITE_BLOCK), SITE_BLOCK, upds_lds<double, 64>(), st>>>(
                g, static_cast<const double2 *>(U0), static_cast<const double2 *>(G), D, partials,
                status);
    };
    if (update_shared64_ok(g)) {
        if (g.ff32) shared(static_cast<float2 *>(Dout));
        else shared(static_cast<double2 *>(Dout));
    } else if (g.ff32) go(k_update_u0<float>, static_cast<float2 *>(Dout));
    else go(k_update_u0<double>, static_cast<double2 *>(Dout));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (fp.enabled) finalize(partials, site_blocks(g.V), status, fp, st);
    return hipGetLastError();
}

hipError_t launch_unpack_rotated(const void *U0, const void *G, double *Uaos, const geom &g,
                                 hipStream_t st) {
    if (!g.keeps_u0()) return hipErrorInvalidValue;
    k_unpack_rotated<<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(
        g, static_cast<const double2 *>(U0), static_cast<const double2 *>(G),
        reinterpret_cast<double2 *>(Uaos));
    return hipGetLastError();
}

template hipError_t launch_update<double>(const geom &, const void *, void *, const void *, void *,
                                          void *, double, bool, void *, double *, dev_status *,
                                          const fin_params &, hipStream_t);
template hipError_t launch_update<float>(const geom &, const void *, void *, const void *, void *,
                                         void *, float, bool, void *, double *, dev_status *,
                                         const fin_params &, hipStream_t);

hipError_t launch_reorder_fields(const geom &g, const double2 *in, long si, double2 *out, long so,
                                 int to_natural, hipStream_t st) {
    k_reorder<<<nblk(g.V, 256), 256, 0, st>>>(g, in, si, out, so, to_natural);
    return hipGetLastError();
}

hipError_t launch_finalize(const double *partials, int nparts, dev_status *status,
                           const fin_params &fp, hipStream_t st) {
    finalize(partials, nparts, status, fp, st);
    return hipGetLastError();
}

hipError_t launch_status_reset(dev_status *status, int hist_base, hipStream_t st) {
    k_status_reset<<<1, 1, 0, st>>>(status, hist_base);
    return hipGetLastError();
}

hipError_t launch_reduce_only(const double *partials, int nparts, double *out2, hipStream_t st) {
    k_reduce_only<<<1, FIN_BLOCK, 0, st>>>(partials, nparts, out2);
    return hipGetLastError();
}

hipError_t launch_measure_finalize(const double *partials, int nparts, double *out, double normF,
                                   double normT, hipStream_t st) {
    k_measure_finalize<<<1, FIN_BLOCK, 0, st>>>(partials, nparts, out, normF, normT);
    return hipGetLastError();
}

hipError_t launch_g_identity(void *G32, const geom &g, hipStream_t st) {
    if (g.nc == 2) return launch_g_identity_su2(G32, g, st);
    k_g_identity<<<nblk(g.V, 256), 256, 0, st>>>(static_cast<float2 *>(G32), g.V, g.S);
    return hipGetLastError();
}

hipError_t launch_switch(const geom &g, const void *G32, const double *U0aos, void *L64,
                         hipStream_t st) {
    if (g.nc == 2) return launch_switch_su2(g, G32, U0aos, L64, st);
    auto Gp = static_cast<const float2 *>(G32);
    auto U0 = reinterpret_cast<const double2 *>(U0aos);
    auto Lp = static_cast<double2 *>(L64);
    if (g.lf == 18) k_switch<18><<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Gp, U0, Lp);
    else if (g.lf == 8) k_switch<8><<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Gp, U0, Lp);
    else k_switch<12><<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Gp, U0, Lp);
    return hipGetLastError();
}

hipError_t launch_switch_div(const geom &g, const void *G32, const double *U0aos, void *L64,
                             void *D, double *partials, dev_status *status, const fin_params &fp,
                             hipStream_t st) {
    if (g.nc != 3) return hipErrorInvalidValue;
    const hipError_t e = with_field_type<double>(g, [&](auto tf) -> hipError_t {
        using TF = decltype(tf);
        auto Gp = static_cast<const float2 *>(G32);
        auto U0 = reinterpret_cast<const double2 *>(U0aos);
        auto Lp = static_cast<double2 *>(L64);
        auto Dp = static_cast<vec2_t<TF> *>(D);
        if (g.lf == 18)
            k_switch_div<18, TF><<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Gp, U0, Lp, Dp, partials);
        else if (g.lf == 8)
            k_switch_div<8, TF><<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Gp, U0, Lp, Dp, partials);
        else
            k_switch_div<12, TF><<<site_blocks(g.V), SITE_BLOCK, 0, st>>>(g, Gp, U0, Lp, Dp, partials);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    if (fp.enabled) finalize(partials, site_blocks(g.V), status, fp, st);
    return hipGetLastError();
}

hipError_t launch_field_from_matrix(const double *Maos, void *D64, long V, long S, hipStream_t st) {
    k_field_from_matrix<<<nblk(V, 256), 256, 0, st>>>(reinterpret_cast<const double2 *>(Maos),
                                                      static_cast<double2 *>(D64), V, S);
    return hipGetLastError();
}

hipError_t launch_matrix_from_field(const void *D64, double *Maos, long V, long S, hipStream_t st) {
    k_matrix_from_field<<<nblk(V, 256), 256, 0, st>>>(static_cast<const double2 *>(D64),
                                                      reinterpret_cast<double2 *>(Maos), V, S);
    return hipGetLastError();
}

}  // namespace lgf
