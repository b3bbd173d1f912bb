// Device helpers shared by the kernel translation units.
#pragma once
#include "fft.hpp"
#include "kernels.hpp"
#include "su3.hpp"

namespace lgf {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

// Blocks are dispatched round-robin over the 8 XCDs; map them so that each
// XCD (own L2) walks a contiguous range of sites and neighbour data is shared.
__device__ __forceinline__ int xcd_block(int b, int nb) {
    const int q = nb >> 3, r = nb & 7, x = b & 7, k = b >> 3;
    return x * q + (x < r ? x : r) + k;
}

// Site of thread tid of site-kernel block b.  Blocks are first remapped so
// that each XCD walks a contiguous range.
//   g.tblock == 0: consecutive sites.
//   g.tblock == 1: the block's four waves take 64 consecutive xy-sites (a
//     "segment", one coalesced row each) at 4 consecutive t.  Blocks advance
//     through a group of g.sgroup adjacent segments fastest, then z, then the
//     segment group, then t: three of four t-neighbour pairs are inside a
//     block, and the blocks holding the y and z neighbours are at most
//     g.sgroup positions apart in dispatch order on the same XCD, so their
//     lines are still in that XCD's L2.  When each XCD's range holds
//     g.tslab > 1 slices of 4 t, the slices are walked inside z (after the
//     segment group), so the t neighbours across two slices of one XCD are
//     g.sgroup positions apart too instead of a whole slice.
__device__ __forceinline__ long block_site(const geom &g, int b, int nb, int tid) {
    const int B = xcd_block(b, nb);
    if (!g.tblock) return (long)B * SITE_BLOCK + tid;
    const int Lxy = g.Lx * g.Ly, G = g.sgroup, ngrp = (Lxy >> 6) / G;
    const int sg = B % G;
    int r = B / G;
    const int sl = r % g.tslab;
    r /= g.tslab;
    const int z = r % g.Lz;
    r /= g.Lz;
    const int slab = (r / ngrp) * g.tslab + sl;
    const int seg = (r % ngrp) * G + sg, t = slab * 4 + (tid >> 6);
    return (long)seg * 64 + (tid & 63) + (long)Lxy * (z + (long)g.Lz * t);
}

struct nbr {
    long p[4], m[4];  // s + mu, s - mu (periodic)
};

// Site coordinates in 32-bit unsigned arithmetic (every supported volume,
// up to 128^4 sites, is below 2^31).
__device__ __forceinline__ nbr neighbours(const geom &g, long s) {
    nbr n;
    unsigned r = (unsigned)s;
    const unsigned Lx = g.Lx, Ly = g.Ly, Lz = g.Lz;
    unsigned q = r / Lx;
    const int x = (int)(r - q * Lx);
    r = q; q = r / Ly;
    const int y = (int)(r - q * Ly);
    r = q; q = r / Lz;
    const int z = (int)(r - q * Lz);
    const int t = (int)q;
    const long sy = g.Lx, sz = (long)g.Lx * g.Ly, stt = sz * g.Lz;
    n.p[0] = (x == g.Lx - 1) ? s - (g.Lx - 1) : s + 1;
    n.m[0] = (x == 0) ? s + (g.Lx - 1) : s - 1;
    n.p[1] = (y == g.Ly - 1) ? s - (long)(g.Ly - 1) * sy : s + sy;
    n.m[1] = (y == 0) ? s + (long)(g.Ly - 1) * sy : s - sy;
    n.p[2] = (z == g.Lz - 1) ? s - (long)(g.Lz - 1) * sz : s + sz;
    n.m[2] = (z == 0) ? s + (long)(g.Lz - 1) * sz : s - sz;
    n.p[3] = (t == g.Lt - 1) ? s - (long)(g.Lt - 1) * stt : s + stt;
    n.m[3] = (t == 0) ? s + (long)(g.Lt - 1) * stt : s - stt;
    return n;
}

// Deterministic block sum of two doubles into partials[2*slot + {0,1}].
template <int NT>
__device__ __forceinline__ void block_sum2(double a, double b, double *partials, int slot) {
    static_assert(NT % 64 == 0, "wave64 blocks");
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
    if (threadIdx.x == 0) {
        double A = 0, B = 0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) {
            A += sa[i];
            B += sb[i];
        }
        partials[2 * slot] = A;
        partials[2 * slot + 1] = B;
    }
}

// ---------------------------------------------------------------------------
// fixed-order sum of block partials and the stopping test
// ---------------------------------------------------------------------------

template <int NT>
__device__ __forceinline__ void fixed_order_sum(const double *__restrict__ partials, int nparts,
                                                double &A, double &B) {
    // thread t adds pairs t, t + NT, t + 2 NT, ... in that order; four 16-byte
    // loads are in flight per step
    const double2 *p2 = reinterpret_cast<const double2 *>(partials);
    double a = 0, b = 0;
    int i = threadIdx.x;
    for (; i + 3 * NT < nparts; i += 4 * NT) {
        const double2 v0 = p2[i], v1 = p2[i + NT], v2 = p2[i + 2 * NT], v3 = p2[i + 3 * NT];
        a += v0.x;
        b += v0.y;
        a += v1.x;
        b += v1.y;
        a += v2.x;
        b += v2.y;
        a += v3.x;
        b += v3.y;
    }
    for (; i < nparts; i += NT) {
        const double2 v = p2[i];
        a += v.x;
        b += v.y;
    }
    __shared__ double sa[NT], sb[NT];
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int h = NT / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            sa[threadIdx.x] += sa[threadIdx.x + h];
            sb[threadIdx.x] += sb[threadIdx.x + h];
        }
        __syncthreads();
    }
    A = sa[0];
    B = sb[0];
}

// The same without a block-wide tree: lane l of 64 adds pairs l, l + 64, ...,
// then the lanes are added pairwise, in every wave, without LDS or barriers.
// For a few hundred pairs; the same bits in every thread of every block,
// whatever its size: the stopping test of a sweep is taken by kernels of
// different block sizes.  ODD_BLOCKS: also in blocks that are no multiple of a
// wave; their first wave does it, or, below 64 threads, every thread stands for
// several lanes, in LDS.
template <bool ODD_BLOCKS = false>
__device__ __forceinline__ void wave_sum(const double *__restrict__ partials, int nparts, double &A,
                                         double &B) {
    const double2 *p2 = reinterpret_cast<const double2 *>(partials);
    // four loads in flight; beyond the last pair +0 is added, which changes no sum
    auto lane_sum = [&](int lane) {
        double2 r = make_double2(0, 0);
        for (int i = lane; i < nparts; i += 256) {
            double2 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = p2[min(i + 64 * k, nparts - 1)];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                r.x += i + 64 * k < nparts ? v[k].x : 0.0;
                r.y += i + 64 * k < nparts ? v[k].y : 0.0;
            }
        }
        return r;
    };
    const bool whole = !ODD_BLOCKS || blockDim.x % 64 == 0;
    double2 r = make_double2(0, 0);
    if (whole || (blockDim.x > 64 && threadIdx.x < 64)) {
        r = lane_sum(threadIdx.x & 63);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            r.x += __shfl_down(r.x, off);
            r.y += __shfl_down(r.y, off);
        }
        r.x = __shfl(r.x, 0);
        r.y = __shfl(r.y, 0);
    }
    if constexpr (ODD_BLOCKS) {
        if (!whole) {
            __shared__ double2 v[64];
            if (blockDim.x > 64) {
                if (threadIdx.x == 0) v[0] = r;
            } else {
                for (int l = threadIdx.x; l < 64; l += blockDim.x) v[l] = lane_sum(l);
                for (int off = 32; off > 0; off >>= 1) {
                    __syncthreads();
                    for (int l = threadIdx.x; l < off; l += blockDim.x) {
                        v[l].x += v[l + off].x;
                        v[l].y += v[l + off].y;
                    }
                }
            }
            __syncthreads();
            r = v[0];
        }
    }
    A = r.x;
    B = r.y;
}

// The state after a sweep whose partials sum to A and B: F = A normF, theta =
// B normT, and the stopping test.  write_hist: also the history (one thread).
__device__ __forceinline__ dev_status next_state(double A, double B, dev_status st,
                                                 const fin_params &fp, bool write_hist = true) {
    const double F = A * fp.normF, th = B * fp.normT;
    if (fp.increment) st.n += 1;
    const int h = st.hist_base + st.n;
    if (write_hist && h < fp.hist_cap) {
        fp.histF[h] = F;
        fp.histT[h] = th;
    }
    st.F = F;
    st.theta = th;
    if (!isfinite(th) || !isfinite(F)) {
        st.done = 1;
        st.code = ST_NONFINITE;
    } else if (th < fp.tol) {
        st.done = 1;
        st.code = ST_CONVERGED;
    } else if (st.n >= fp.max_iter) {
        st.done = 1;
        st.code = ST_MAXITER;
    } else if (fp.tol > 0) {
        // a solve (tol > 0) also stops when theta diverges or stalls; a fixed
        // count of sweeps (tol == 0) runs them all
        st.rises = (st.n > 0 && th > st.theta_prev) ? st.rises + 1 : 0;
        st.since_min = (st.n == 0 || th < st.theta_min) ? 0 : st.since_min + 1;
        if (st.rises >= DIVERGE_RISES && th > DIVERGE_GROWTH * st.theta_min) {
            st.done = 1;
            st.code = ST_DIVERGING;
        } else if (fp.stall > 0 && st.since_min >= fp.stall) {
            st.done = 1;
            st.code = ST_STALLED;
        }
    }
    st.theta_prev = th;
    st.theta_min = (st.n == 0 || th < st.theta_min) ? th : st.theta_min;
    return st;
}

// The start of a sweep's first kernel: whether the sweeps are over, with the
// stopping test of the sweep before if fold asks for it (every wave sums the
// partials; the grid's first thread writes the state).
template <bool ODD_BLOCKS = false>
__device__ __forceinline__ bool sweeps_over(const dev_status *__restrict__ status,
                                            const fold_args &fold) {
    if (!fold.fp.enabled) return status->done != 0;
    const bool first = (threadIdx.x | blockIdx.x | blockIdx.y | blockIdx.z) == 0;
    const dev_status st = *status;
    if (st.done) {
        if (first) *fold.out = st;
        return true;
    }
    double A, B;
    wave_sum<ODD_BLOCKS>(fold.partials, fold.nparts, A, B);
    const dev_status nx = next_state(A, B, st, fold.fp, first);
    if (first) *fold.out = nx;
    return nx.done != 0;
}

// Lattices whose sweep kernels load their tiles before they look at the state
// (see discard): where a launch is a few microseconds, the state's latency is
// a good part of it; where it is not, a sweep enqueued past the stop should
// return without reading its field.
__device__ __forceinline__ bool tiles_first(const geom &g) { return g.V <= 163840; }

// A use of loaded values on the path that returns without them: it keeps the
// loads above the branch, so that their latency overlaps that of the state the
// branch depends on.
template <class T, int N> __device__ __forceinline__ void discard(const cpx<T> (&a)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" ::"v"(a[j].re), "v"(a[j].im));
}

}  // namespace lgf
