// Small lattices: the whole accelerated transform of a field in one block.
#include <algorithm>

#include "fft_kernels.hpp"

namespace lgf {

// A sweep of a small lattice is a chain of launches of a few microseconds each
// (8^4: (x,y) 3.6, (z,t) 4.5, (x,y) 3.4, stopping test 3.1 and the gaps
// between them), whatever little they move.  Here one block holds a whole
// field in LDS, rows of Lx padded by one element, and runs the forward
// transforms, the scaling and the inverse transforms along all four axes; the
// stopping test of the sweep before rides along (sweeps_over).  The axes come in the order of the general passes (small_plan), so each value
// goes through the same operations.
template <class T, int RMAX, int NTHR>
__global__ void __launch_bounds__(NTHR)
    k_fft4_small(geom g, vec2_t<T> *__restrict__ D, const vec2_t<T> *__restrict__ tw,
                 const T *__restrict__ ptab, T p2max_over_V, small_plan sp,
                 const dev_status *__restrict__ status, fold_args fold) {
    extern __shared__ unsigned char smem_raw[];
    vec2_t<T> *lds = reinterpret_cast<vec2_t<T> *>(smem_raw);
    const int Lx = g.Lx, P = Lx + 1, V = (int)g.V;
    vec2_t<T> *F = D + (long)blockIdx.x * g.S;
    // twiddles in LDS behind the field: a table read per axis would wait for
    // memory in every one of the seven transforms
    vec2_t<T> *twl = lds + (V / Lx) * P;
    const int nt = Lx + g.Ly + g.Lz + g.Lt;
    for (int i = threadIdx.x; i < nt; i += NTHR) twl[i] = tw[i];
    for (int i = threadIdx.x; i < V; i += NTHR) {
        const int r = i / Lx;
        lds[i + r] = F[i];  // row r starts at r P
    }
    if (sweeps_over(status, fold)) return;
    __syncthreads();
    auto axis_base = [&](int ax) {
        const int xd = ax == 0 ? 1 : Lx;
        const int M = ax == 0 ? V : ax == 1 ? 1 : ax == 2 ? g.Ly : g.Ly * g.Lz;
        const int Q = ax == 1 ? P * g.Ly : ax == 2 ? P * g.Ly * g.Lz : 0;
        // column c: x fastest (none for the x axis), then the rows it starts at
        return [=](int c) {
            const int r = c / xd, m = r / M;
            return (c - r * xd) + (r - m * M) * P + m * Q;
        };
    };
    auto extent = [&](int ax) { return ax == 0 ? Lx : ax == 1 ? g.Ly : ax == 2 ? g.Lz : g.Lt; };
    auto stride = [&](int ax) {
        return ax == 0 ? 1 : ax == 1 ? P : ax == 2 ? P * g.Ly : P * g.Ly * g.Lz;
    };
    auto table = [&](int ax) {
        return ax == 0 ? 0 : ax == 1 ? Lx : ax == 2 ? Lx + g.Ly : Lx + g.Ly + g.Lz;
    };
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const int ax = sp.order[k], n = extent(ax);
        lds_axis_fft<-1, T, RMAX>(n, lds, V / n, stride(ax), axis_base(ax), twl + table(ax));
        __syncthreads();
    }
    {
        // the innermost axis (z or t): p2 of a column without its term, summed
        // as (x + y) + the other one
        const int ax = sp.order[3], n = extent(ax), ot = ax == 2 ? 3 : 2;
        const T *px = ptab, *py = ptab + table(1), *po = ptab + table(ot), *pa = ptab + table(ax);
        const int Ly = g.Ly;
        auto prep = [=](int c) -> T {
            const int x = c % Lx, r = c / Lx;
            return (px[x] + py[r % Ly]) + po[r / Ly];
        };
        auto scale = [=](T b, int k) -> T { return fa_factor<T>(b, pa[k], p2max_over_V); };
        lds_axis_fsi<T, RMAX>(n, lds, V / n, stride(ax), axis_base(ax), prep, scale, twl + table(ax));
        __syncthreads();
    }
#pragma unroll 1
    for (int k = 2; k >= 0; --k) {
        const int ax = sp.order[k], n = extent(ax);
        lds_axis_fft<1, T, RMAX>(n, lds, V / n, stride(ax), axis_base(ax), twl + table(ax));
        __syncthreads();
    }
    for (int i = threadIdx.x; i < V; i += NTHR) {
        const int r = i / Lx;
        F[i] = lds[i + r];
    }
}

constexpr int SMALL_THREADS_16 = 1024, SMALL_THREADS_32 = 512;
// rows of two sites pad the most, and no four extents of so few sites add up to
// more than 256 + 2 + 2 + 2 twiddles
static_assert((SMALL_MAX_SITES / 2 * 3 + 262) * sizeof(double2) <= 64 * 1024,
              "LDS of a field beyond what a launch gets without an attribute");

template <class T> small_plan plan_small(const geom &g, const fft_plan &p) {
    small_plan s;
    const size_t lds = ((size_t)(g.V / g.Lx) * (g.Lx + 1) + g.Lx + g.Ly + g.Lz + g.Lt) * sizeof(vec2_t<T>);
    if (g.V > SMALL_MAX_SITES) return s;
    s.on = true;
    s.lds = lds;
    s.rmax = std::max(std::max(fft_tier(g.Lx), fft_tier(g.Ly)), std::max(fft_tier(g.Lz), fft_tier(g.Lt)));
    // the order of the general passes: (x,t) planes take x, t and the (y,z)
    // tiles y, z; register columns take their column's axis first and scale
    // inside z, the one-axis passes inside t; whole planes take x first
    if (p.t2) {
        s.order[0] = 0;
        s.order[1] = 3;
        s.order[2] = 1;
        s.order[3] = 2;
    } else {
        s.order[0] = p.xy == 0 ? 1 : 0;
        s.order[1] = p.xy == 0 ? 0 : 1;
        s.order[2] = p.rc ? 3 : 2;
        s.order[3] = p.rc ? 2 : 3;
    }
    return s;
}

template <class T>
hipError_t launch_fft4_small(const geom &g, void *D, const void *tw, const T *ptab, T p2max_over_V,
                             const small_plan &sp, const dev_status *status, const fold_args &fold,
                             hipStream_t st) {
    if (!sp.on) return hipErrorInvalidValue;
    auto Dp = static_cast<vec2_t<T> *>(D);
    auto twp = static_cast<const vec2_t<T> *>(tw);
    if (sp.rmax <= 16)
        k_fft4_small<T, 16, SMALL_THREADS_16><<<g.nf, SMALL_THREADS_16, sp.lds, st>>>(
            g, Dp, twp, ptab, p2max_over_V, sp, status, fold);
    else
        k_fft4_small<T, 32, SMALL_THREADS_32><<<g.nf, SMALL_THREADS_32, sp.lds, st>>>(
            g, Dp, twp, ptab, p2max_over_V, sp, status, fold);
    return hipGetLastError();
}

#define LGF_SMALL(T)                                                                              \
    template small_plan plan_small<T>(const geom &, const fft_plan &);                            \
    template hipError_t launch_fft4_small<T>(const geom &, void *, const void *, const T *, T,    \
                                             const small_plan &, const dev_status *,              \
                                             const fold_args &, hipStream_t);
LGF_SMALL(double)
LGF_SMALL(float)
#undef LGF_SMALL

}  // namespace lgf
