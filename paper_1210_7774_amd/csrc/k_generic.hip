// Per-point level kernels for any dimension (1, 2, 3): red-black half
// sweeps, weighted Jacobi, residual + full-weighting restriction, bilinear /
// trilinear prolongation + correction, and the FP64 residual norm with the
// device-side stop test.  They serve the 3D levels, the Jacobi smoother and
// the outer residual of iterative refinement; the 2D Gauss-Seidel levels use
// the fused row-marching kernels.
//
// Grid convention: 1-based interior index (i, j, k), x fastest, element at
// (i-1) + (j-1) pitch + (k-1) ppitch; values outside [1, n] are the Dirichlet
// zeros.  Nodal coefficients (2D) cover (n+2)^2 nodes.
#include "dev_common.h"

namespace mgx {

template <int DIM>
struct Idx {
    int n;
    long long pitch, ppitch;
    __device__ __forceinline__ long long off(int i, int j, int k) const
    {
        return (long long)(i - 1) + (DIM > 1 ? (long long)(j - 1) * pitch : 0) +
               (DIM > 2 ? (long long)(k - 1) * ppitch : 0);
    }
    __device__ __forceinline__ bool in(int i, int j, int k) const
    {
        return i >= 1 && i <= n && (DIM < 2 || (j >= 1 && j <= n)) && (DIM < 3 || (k >= 1 && k <= n));
    }
};

template <class S, int DIM>
__device__ __forceinline__ typename Traits<S>::C getu(const S *u, const Idx<DIM> &x, int i, int j, int k)
{
    using C = typename Traits<S>::C;
    if (!u || !x.in(i, j, k)) return (C)0;
    return Traits<S>::ld(u + x.off(i, j, k));
}

template <class C>
__device__ __forceinline__ C harm(C a, C b)
{
    return (C)2 * a * b / (a + b);
}

// Faces of the 2D variable-coefficient operator at node (i, j):
// west, east, south (row j-1), north (row j+1).
template <class C>
__device__ __forceinline__ void faces2d(const C *a, int n, int i, int j, C &ww, C &we, C &ws, C &wn)
{
    const long long s = n + 2;
    const C ac = a[i + s * j];
    ww = harm(ac, a[(i - 1) + s * j]);
    we = harm(ac, a[(i + 1) + s * j]);
    ws = harm(ac, a[i + s * (j - 1)]);
    wn = harm(ac, a[i + s * (j + 1)]);
}

// Gauss-Seidel point value from the current neighbours.
template <class S, class F, int DIM, bool VC>
__device__ __forceinline__ typename Traits<S>::C relax_pt(const S *u, const F *f, const typename Traits<S>::C *a,
                                                          const Idx<DIM> &x, double h2d, int i, int j, int k)
{
    using C = typename Traits<S>::C;
    const C h2 = (C)h2d;
    const C fv = (C)f[x.off(i, j, k)];
    if constexpr (!VC) {
        C s = h2 * fv;
        s = s + getu(u, x, i - 1, j, k);
        s = s + getu(u, x, i + 1, j, k);
        if (DIM > 1) {
            s = s + getu(u, x, i, j - 1, k);
            s = s + getu(u, x, i, j + 1, k);
        }
        if (DIM > 2) {
            s = s + getu(u, x, i, j, k - 1);
            s = s + getu(u, x, i, j, k + 1);
        }
        return s * (C)(DIM == 1 ? 0.5 : DIM == 2 ? 0.25 : 1.0 / 6.0);
    } else {
        C ww, we, ws, wn;
        faces2d(a, x.n, i, j, ww, we, ws, wn);
        C s = h2 * fv;
        s = s + ww * getu(u, x, i - 1, j, k);
        s = s + we * getu(u, x, i + 1, j, k);
        s = s + ws * getu(u, x, i, j - 1, k);
        s = s + wn * getu(u, x, i, j + 1, k);
        return s / (((ww + we) + ws) + wn);
    }
}

// (A u) at one point.
template <class S, int DIM, bool VC>
__device__ __forceinline__ typename Traits<S>::C apply_pt(const S *u, const typename Traits<S>::C *a,
                                                          const Idx<DIM> &x, double ih2d, int i, int j, int k)
{
    using C = typename Traits<S>::C;
    const C uc = getu(u, x, i, j, k);
    C s;
    if constexpr (!VC) {
        s = (uc - getu(u, x, i - 1, j, k)) + (uc - getu(u, x, i + 1, j, k));
        if (DIM > 1) s = (s + (uc - getu(u, x, i, j - 1, k))) + (uc - getu(u, x, i, j + 1, k));
        if (DIM > 2) s = (s + (uc - getu(u, x, i, j, k - 1))) + (uc - getu(u, x, i, j, k + 1));
    } else {
        C ww, we, ws, wn;
        faces2d(a, x.n, i, j, ww, we, ws, wn);
        s = ((ww * (uc - getu(u, x, i - 1, j, k)) + we * (uc - getu(u, x, i + 1, j, k))) +
             ws * (uc - getu(u, x, i, j - 1, k))) +
            wn * (uc - getu(u, x, i, j + 1, k));
    }
    return s * (C)ih2d;
}

__device__ __forceinline__ void coords(long long p, int n, int dim, int &i, int &j, int &k)
{
    i = (int)(p % n) + 1;
    p /= n;
    j = 1;
    k = 1;
    if (dim > 1) {
        j = (int)(p % n) + 1;
        p /= n;
    }
    if (dim > 2) k = (int)p + 1;
}

__host__ __device__ __forceinline__ long long npts(int n, int dim)
{
    long long m = n;
    if (dim > 1) m *= n;
    if (dim > 2) m *= n;
    return m;
}

// ---- red-black half sweep (in place on B; colours are disjoint) -------------
template <class S, class F, int DIM, bool VC>
__global__ __launch_bounds__(256) void k_rb_half(GenArgs g)
{
    using C = typename Traits<S>::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<DIM> x{L.n, L.pitch, L.ppitch};
    S *u = (S *)L.B;
    const F *f = (const F *)L.f;
    const C *a = (const C *)L.a;
    // thread p handles the pair of x-points (2m+1, 2m+2) and updates the one of the colour
    const int half = (L.n + 1) / 2;
    long long total = (long long)half * (DIM > 1 ? L.n : 1) * (DIM > 2 ? L.n : 1);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < total;
         p += (long long)gridDim.x * blockDim.x) {
        long long t = p;
        const int m = (int)(t % half);
        t /= half;
        int j = 1, k = 1;
        if (DIM > 1) {
            j = (int)(t % L.n) + 1;
            t /= L.n;
        }
        if (DIM > 2) k = (int)t + 1;
        int i = 2 * m + 1;
        if (((i + (DIM > 1 ? j : 0) + (DIM > 2 ? k : 0)) & 1) != g.colour) i += 1;
        if (i > L.n) continue;
        C v = relax_pt<S, F, DIM, VC>(u, f, a, x, L.h2, i, j, k);
        Traits<S>::st(u + x.off(i, j, k), Traits<S>::rnd(v));
    }
}

// ---- weighted Jacobi (out of place): dst = src + omega D^-1 (f - A src) -------
template <class S, class F, int DIM, bool VC>
__global__ __launch_bounds__(256) void k_jacobi(GenArgs g)
{
    using C = typename Traits<S>::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<DIM> x{L.n, L.pitch, L.ppitch};
    const S *src = g.u_zero ? nullptr : (const S *)g.src;
    S *dst = (S *)g.dst;
    const F *f = (const F *)L.f;
    const C *a = (const C *)L.a;
    const long long m = npts(L.n, DIM);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(p, L.n, DIM, i, j, k);
        const C uc = getu(src, x, i, j, k);
        const C r = (C)f[x.off(i, j, k)] - apply_pt<S, DIM, VC>(src, a, x, L.inv_h2, i, j, k);
        C diag;
        if constexpr (!VC) {
            diag = (C)(2 * DIM) * (C)L.inv_h2;
        } else {
            C ww, we, ws, wn;
            faces2d(a, L.n, i, j, ww, we, ws, wn);
            diag = (((ww + we) + ws) + wn) * (C)L.inv_h2;
        }
        Traits<S>::st(dst + x.off(i, j, k), Traits<S>::rnd(uc + (C)g.omega * r / diag));
    }
}

// ---- residual + full weighting: fc(I) = sum_o w(o) r(2I + o) / 4^d ---------------
template <class S, class F>
__global__ __launch_bounds__(256) void k_resid_restrict1(GenArgs g)
{
    using C = typename Traits<S>::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<1> x{L.n, L.pitch, L.ppitch};
    const S *u = (const S *)L.B;
    const F *f = (const F *)L.f;
    F *fc = (F *)L.fc;
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < L.nc; p += gridDim.x * blockDim.x) {
        C s = (C)0;
        for (int ox = -1; ox <= 1; ++ox) {
            const int i = 2 * (p + 1) + ox;
            const C r = (C)f[i - 1] - apply_pt<S, 1, false>(u, nullptr, x, L.inv_h2, i, 1, 1);
            s = s + (C)(2 - (ox < 0 ? -ox : ox)) * r;
        }
        fc[p] = (F)(s * (C)0.25);
    }
}

// 2D: a wavefront takes 64 fine columns (30 coarse points of them) and kRRows
// coarse rows, all loads in flight at once; the neighbours' values, their faces
// and residuals come from the next lanes, so each residual and each face is
// computed once or twice instead of 2.25 times (a coarse point by itself takes
// nine residuals of five points and their 36 faces: 1023^2 variable-coefficient
// FP32 13.2 us -> 6.4).  The sums and their order are those of the 1D kernel
// above, rows from below, west to east.
constexpr int kRRows = 4;
template <class S, class F, bool VC>
__global__ __launch_bounds__(256) void k_resid_restrict2(GenArgs g)
{
    using T = Traits<S>;
    using C = typename T::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    const int n = L.n, nc = L.nc, lane = threadIdx.x & 63;
    const int strips = (nc + 29) / 30;
    const long long unit = blockIdx.x * 4LL + (threadIdx.x >> 6);
    const int I0 = 30 * (int)(unit % strips), J0 = kRRows * (int)(unit / strips);
    if (J0 >= nc) return;
    const S *ub = (const S *)L.B;
    const F *fb = (const F *)L.f;
    const C *a = (const C *)L.a;
    constexpr int NR = 2 * kRRows + 3;  // fine rows 2 J0 .. 2 J0 + NR - 1
    const int i = 2 * I0 + lane;        // this lane's fine column; the even lanes 2 .. 60 hold coarse ones
    const bool cin = i >= 1 && i <= n;
    C u[NR], f[NR], an[VC ? NR : 1];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const int j = 2 * J0 + q;
        const bool in = cin && j >= 1 && j <= n, fin = q > 0 && q < NR - 1;
        if constexpr (sizeof(C) == 8) {
            u[q] = in ? T::ld(ub + (long long)(j - 1) * L.pitch + (i - 1)) : (C)0;
            f[q] = in && fin ? (C)gld(fb + (long long)(j - 1) * L.pitch + (i - 1)) : (C)0;
        } else {
            // 4- and 2-byte loads at clamped places, selected below: under a
            // condition they wait for one another (511^2 FP32 7.7 -> 6.7 us, bfloat16
            // 9.9 -> 6.7; FP64 with coefficients 6.8 -> 7.2, so not there)
            const long long o = (long long)(min(max(j, 1), n) - 1) * L.pitch + (min(max(i, 1), n) - 1);
            u[q] = T::ld(ub + o);
            f[q] = fin ? (C)gld(fb + o) : (C)0;
        }
        if constexpr (VC) an[q] = gld(a + (long long)min(j, n + 1) * (n + 2) + min(i, n + 1));
    }
    if constexpr (sizeof(C) == 4) {
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int j = 2 * J0 + q;
            const bool in = cin && j >= 1 && j <= n;
            u[q] = in ? u[q] : (C)0;
            f[q] = in ? f[q] : (C)0;
        }
    }
    C ws = (C)0, acc = (C)0;
    if constexpr (VC) ws = harm(an[1], an[0]);
    F *fc = (F *)L.fc;
#pragma unroll
    for (int q = 1; q < NR - 1; ++q) {
        const C uc = u[q], w = from_prev(uc), e = from_next(uc);
        C s;
        if constexpr (!VC) {
            s = (uc - w) + (uc - e);
            s = (s + (uc - u[q - 1])) + (uc - u[q + 1]);
        } else {
            const C we = harm(an[q], from_next(an[q])), ww = from_prev(we), wn = harm(an[q], an[q + 1]);
            s = ((ww * (uc - w) + we * (uc - e)) + ws * (uc - u[q - 1])) + wn * (uc - u[q + 1]);
            ws = wn;
        }
        const C r = f[q] - s * (C)L.inv_h2, rl = from_prev(r), rr = from_next(r);
        if (q % 2 == 0) {  // the coarse point's own row
            acc = acc + (C)2 * rl;
            acc = acc + (C)4 * r;
            acc = acc + (C)2 * rr;
            continue;
        }
        if (q > 1) {  // the row above it
            acc = acc + rl;
            acc = acc + (C)2 * r;
            acc = acc + rr;
            const int I = I0 + lane / 2, J = J0 + q / 2;
            if (!(lane & 1) && lane >= 2 && lane <= 60 && I <= nc && J <= nc)
                gst(fc + (long long)(J - 1) * L.cpitch + (I - 1), (F)(acc * (C)0.0625));
        }
        acc = rl;  // the row below the next
        acc = acc + (C)2 * r;
        acc = acc + rr;
    }
}

// 3D in two streaming passes: the fused form recomputes 27 fine residuals of
// 7 points each per coarse point.  Pass 1 writes r = f - A u (compute type,
// contiguous) into the level's spare state buffer A; pass 2 applies the
// same weights in the same order, so the coarse values are unchanged.
template <class S, class F, int DIM, bool VC>
__global__ __launch_bounds__(256) void k_residual_to_a(GenArgs g)
{
    using C = typename Traits<S>::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<DIM> x{L.n, L.pitch, L.ppitch};
    const S *u = (const S *)L.B;
    const F *f = (const F *)L.f;
    const C *a = (const C *)L.a;
    C *r = (C *)L.A;
    const long long m = npts(L.n, DIM);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(p, L.n, DIM, i, j, k);
        r[p] = (C)f[x.off(i, j, k)] - apply_pt<S, DIM, VC>(u, a, x, L.inv_h2, i, j, k);
    }
}

// 3D pass 1 as column marches (the vertical neighbours stay in registers)
template <class S, class F>
__global__ __launch_bounds__(256) void k_residual_to_a3(GenArgs g)
{
    using T = Traits<S>;
    using C = typename T::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<3> x{L.n, L.pitch, L.ppitch};
    const int n = L.n;
    const S *u = (const S *)L.B;
    const F *f = (const F *)L.f;
    C *r = (C *)L.A;
    const C ih2 = (C)L.inv_h2;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int ntx = (n + 63) / 64, nty = (n + 3) / 4, ntz = (n + 31) / 32;
    const long long nunits = (long long)ntx * nty * ntz;
    auto U = [&](int i, int j, int k) -> C {
        return (i >= 1 && i <= n && j >= 1 && j <= n && k >= 1 && k <= n) ? (C)T::ld(u + x.off(i, j, k)) : (C)0;
    };
    for (long long un = blockIdx.x; un < nunits; un += gridDim.x) {
        const int i = (int)(un % ntx) * 64 + tx + 1, j = (int)((un / ntx) % nty) * 4 + ty + 1;
        const int k0 = (int)(un / ((long long)ntx * nty)) * 32 + 1, k1 = min(k0 + 32, n + 1);
        if (i > n || j > n) continue;
        C dn = U(i, j, k0 - 1), c = U(i, j, k0);
#pragma unroll 4
        for (int k = k0; k < k1; ++k) {
            const C up = U(i, j, k + 1);
            C sa = (c - U(i - 1, j, k)) + (c - U(i + 1, j, k));
            sa = (sa + (c - U(i, j - 1, k))) + (c - U(i, j + 1, k));
            sa = (sa + (c - dn)) + (c - up);
            r[(long long)(i - 1) + (long long)n * ((j - 1) + (long long)n * (k - 1))] =
                (C)f[x.off(i, j, k)] - sa * ih2;
            dn = c;
            c = up;
        }
    }
}

template <class S, class F, int DIM>
__global__ __launch_bounds__(256) void k_restrict_from_a(GenArgs g)
{
    using C = typename Traits<S>::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<DIM> xc{L.nc, L.cpitch, L.cppitch};
    const C *r = (const C *)L.A;
    F *fc = (F *)L.fc;
    const int n = L.n;
    const long long mc = npts(L.nc, DIM);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < mc;
         p += (long long)gridDim.x * blockDim.x) {
        int I, J, K;
        coords(p, L.nc, DIM, I, J, K);
        C s = (C)0;
        for (int oz = (DIM > 2 ? -1 : 0); oz <= (DIM > 2 ? 1 : 0); ++oz)
            for (int oy = (DIM > 1 ? -1 : 0); oy <= (DIM > 1 ? 1 : 0); ++oy)
                for (int ox = -1; ox <= 1; ++ox) {
                    const int i = 2 * I + ox, j = DIM > 1 ? 2 * J + oy : 1, k = DIM > 2 ? 2 * K + oz : 1;
                    const int wt = (2 - (ox < 0 ? -ox : ox)) * (DIM > 1 ? (2 - (oy < 0 ? -oy : oy)) : 1) *
                                   (DIM > 2 ? (2 - (oz < 0 ? -oz : oz)) : 1);
                    const C rv = r[(long long)(i - 1) + (long long)n * ((j - 1) + (long long)n * (k - 1))];
                    s = s + (C)wt * rv;
                }
        fc[xc.off(I, J, K)] = (F)(s * (C)(DIM == 1 ? 0.25 : DIM == 2 ? 0.0625 : 0.015625));
    }
}

// 3D prolongation + correction as column marches: a thread keeps the
// bilinear (x, y) interpolation of the coarse planes K and K + 1 of its column
// in registers, so each coarse plane is interpolated once per fine column
// instead of once per fine point; the interpolation order is the generic
// kernel's (x, then y, then z)
template <class S>
__global__ __launch_bounds__(256) void k_prolong_correct3(GenArgs g)
{
    using T = Traits<S>;
    using C = typename T::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<3> x{L.n, L.pitch, L.ppitch};
    Idx<3> xc{L.nc, L.cpitch, L.cppitch};
    const int n = L.n;
    S *u = (S *)L.B;
    const S *uc = (const S *)L.Bc;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int ntx = (n + 63) / 64, nty = (n + 3) / 4, ntz = (n + 31) / 32;
    const long long nunits = (long long)ntx * nty * ntz;
    for (long long un = blockIdx.x; un < nunits; un += gridDim.x) {
        const int i = (int)(un % ntx) * 64 + tx + 1, j = (int)((un / ntx) % nty) * 4 + ty + 1;
        const int k0 = (int)(un / ((long long)ntx * nty)) * 32 + 1, k1 = min(k0 + 32, n + 1);
        if (i > n || j > n) continue;
        const int i0 = i / 2, i1 = (i & 1) ? i0 + 1 : i0;
        const int j0 = j / 2, j1 = (j & 1) ? j0 + 1 : j0;
        auto plane = [&](int kk) -> C {
            auto line = [&](int jj) -> C {
                const C a0 = getu(uc, xc, i0, jj, kk);
                return (i & 1) ? (a0 + getu(uc, xc, i1, jj, kk)) * (C)0.5 : a0;
            };
            const C b0 = line(j0);
            return (j & 1) ? (b0 + line(j1)) * (C)0.5 : b0;
        };
        int K = k0 / 2;
        C pk = plane(K), pk1 = plane(K + 1);
        for (int k = k0; k < k1; ++k) {
            if (k / 2 != K) {  // advance one coarse plane
                K = k / 2;
                pk = pk1;
                pk1 = plane(K + 1);
            }
            const C corr = (k & 1) ? (pk + pk1) * (C)0.5 : pk;
            S *p = u + x.off(i, j, k);
            T::st(p, T::rnd((C)T::ld(p) + corr));
        }
    }
}

// ---- prolongation + correction: B += P Bc ------------------------------------
template <class S>
__global__ __launch_bounds__(256) void k_prolong_correct1(GenArgs g)
{
    using C = typename Traits<S>::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<1> xc{L.nc, L.cpitch, L.cppitch};
    S *u = (S *)L.B;
    const S *uc = (const S *)L.Bc;
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < L.n; p += gridDim.x * blockDim.x) {
        // even index -> one parent (weight 1), odd -> two (1/2 each)
        const int i = p + 1, i0 = i / 2;
        const C a0 = getu(uc, xc, i0, 1, 1);
        const C corr = (i & 1) ? (a0 + getu(uc, xc, i0 + 1, 1, 1)) * (C)0.5 : a0;
        Traits<S>::st(u + p, Traits<S>::rnd(Traits<S>::ld(u + p) + corr));
    }
}

// 2D (ADD), and interpolation alone, B = P Bc: a wavefront takes 64 columns of
// 8 rows, all loads in flight at once; each coarse row is interpolated along x
// once (1023^2 FP32 8.2 us -> 6.1, the index arithmetic of a point by itself
// being most of it; 2047^2 FP64 without the sum 19.4 -> 9.0).  Same order: x,
// then y.
template <class S, bool ADD>
__global__ __launch_bounds__(256) void k_prolong_correct2(GenArgs g)
{
    using T = Traits<S>;
    using C = typename T::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    const int n = L.n, nc = L.nc, strips = (n + 63) / 64;
    const long long unit = blockIdx.x * 4LL + (threadIdx.x >> 6);
    const int i = 64 * (int)(unit % strips) + (int)(threadIdx.x & 63) + 1, j0 = 8 * (int)(unit / strips);
    if (j0 >= n || i > n) return;
    S *u = (S *)L.B + (i - 1);
    const S *uc = (const S *)L.Bc;
    const int i0 = i / 2, i1 = i0 + (i & 1);
    // (loads at clamped places, selected afterwards: a two-byte load under a
    // condition fills half a register and waits for its other half; 255^2
    // bfloat16 8.8 -> 6.5 us, a thread a point 6.4)
    const int c0 = max(i0, 1) - 1, c1 = min(i1, nc) - 1;
    C a[5][2], line[5], v[8];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const S *row = uc + (long long)(min(max(j0 / 2 + q, 1), nc) - 1) * L.cpitch;
        a[q][0] = T::ld(row + c0);
        a[q][1] = T::ld(row + c1);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = ADD ? T::ld(u + (long long)min(j0 + q, n - 1) * L.pitch) : (C)0;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const int J = j0 / 2 + q;
        const bool in = J >= 1 && J <= nc;
        const C a0 = in && i0 >= 1 ? a[q][0] : (C)0, a1 = in && i1 <= nc ? a[q][1] : (C)0;
        line[q] = (i & 1) ? (a0 + a1) * (C)0.5 : a0;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        // row j0 + q + 1: odd rows lie between two coarse ones
        const C corr = q % 2 == 0 ? (line[q / 2] + line[q / 2 + 1]) * (C)0.5 : line[(q + 1) / 2];
        if (j0 + q < n) T::st(u + (long long)(j0 + q) * L.pitch, T::rnd(v[q] + corr));
    }
}

// ---- full multigrid: fc = R f (the rhs carried down by full weighting) -------
template <class F, int DIM>
__global__ __launch_bounds__(256) void k_restrict_rhs(GenArgs g)
{
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<DIM> x{L.n, L.pitch, L.ppitch};
    Idx<DIM> xc{L.nc, L.cpitch, L.cppitch};
    const F *f = (const F *)L.f;
    F *fc = (F *)L.fc;
    const long long mc = npts(L.nc, DIM);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < mc;
         p += (long long)gridDim.x * blockDim.x) {
        int I, J, K;
        coords(p, L.nc, DIM, I, J, K);
        F s = (F)0;
        for (int oz = (DIM > 2 ? -1 : 0); oz <= (DIM > 2 ? 1 : 0); ++oz)
            for (int oy = (DIM > 1 ? -1 : 0); oy <= (DIM > 1 ? 1 : 0); ++oy)
                for (int ox = -1; ox <= 1; ++ox) {
                    const int i = 2 * I + ox, j = DIM > 1 ? 2 * J + oy : 1, k = DIM > 2 ? 2 * K + oz : 1;
                    const int wt = (2 - (ox < 0 ? -ox : ox)) * (DIM > 1 ? (2 - (oy < 0 ? -oy : oy)) : 1) *
                                   (DIM > 2 ? (2 - (oz < 0 ? -oz : oz)) : 1);
                    s = s + (F)wt * f[x.off(i, j, k)];
                }
        fc[xc.off(I, J, K)] = s * (F)(DIM == 1 ? 0.25 : DIM == 2 ? 0.0625 : 0.015625);
    }
}

// ---- full multigrid: B = P Bc (the coarse solution interpolated) ---------------
template <class S, int DIM>
__global__ __launch_bounds__(256) void k_interp(GenArgs g)
{
    using C = typename Traits<S>::C;
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<DIM> x{L.n, L.pitch, L.ppitch};
    Idx<DIM> xc{L.nc, L.cpitch, L.cppitch};
    S *u = (S *)L.B;
    const S *uc = (const S *)L.Bc;
    const long long m = npts(L.n, DIM);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(p, L.n, DIM, i, j, k);
        const int i0 = i / 2, i1 = (i & 1) ? i0 + 1 : i0;
        const int j0 = j / 2, j1 = (j & 1) ? j0 + 1 : j0;
        const int k0 = k / 2, k1 = (k & 1) ? k0 + 1 : k0;
        auto line = [&](int jj, int kk) -> C {
            const C a0 = getu(uc, xc, i0, jj, kk);
            return (i & 1) ? (a0 + getu(uc, xc, i1, jj, kk)) * (C)0.5 : a0;
        };
        auto plane = [&](int kk) -> C {
            if (DIM < 2) return line(1, kk);
            const C b0 = line(j0, kk);
            return (j & 1) ? (b0 + line(j1, kk)) * (C)0.5 : b0;
        };
        C v;
        if (DIM < 3) {
            v = plane(1);
        } else {
            const C c0 = plane(k0);
            v = (k & 1) ? (c0 + plane(k1)) * (C)0.5 : c0;
        }
        Traits<S>::st(u + x.off(i, j, k), Traits<S>::rnd(v));
    }
}

__global__ void k_fill_zero(uint32_t *p, long long nwords)
{
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < nwords; q += (long long)gridDim.x * blockDim.x)
        p[q] = 0u;
}

// the grid points of an array with pitches, without what lies between its rows
__global__ __launch_bounds__(256) void k_zero_points(double *u, int n, int dim, long long pitch, long long ppitch)
{
    const long long m = npts(n, dim);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(p, n, dim, i, j, k);
        u[(long long)(i - 1) + (long long)(j - 1) * pitch + (long long)(k - 1) * ppitch] = 0.0;
    }
}

template <class S, int DIM>
__global__ __launch_bounds__(256) void k_copy_state(GenArgs g, const S *src, S *dst)
{
    if (g.state && g.state->done) return;
    const LevelDesc &L = g.L;
    Idx<DIM> x{L.n, L.pitch, L.ppitch};
    const long long m = npts(L.n, DIM);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(p, L.n, DIM, i, j, k);
        dst[x.off(i, j, k)] = src[x.off(i, j, k)];
    }
}

// ---- FP64 residual norm (+ optional r32 / r64 output) -----------------------------
// (the finish kernel that follows reduces the block partials)
// The block's sums of a 256-thread workgroup into its partial slot.
__device__ __forceinline__ void norm_block_sum(double rr, double ff, double *partials, int slot)
{
    __shared__ double srr[4], sff[4];
    rr = wave_sum(rr);
    ff = wave_sum(ff);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        srr[w] = rr;
        sff[w] = ff;
    }
    __syncthreads();
    if (threadIdx.x < 64) put_partial(partials, slot, ((srr[0] + srr[1]) + srr[2]) + srr[3],
                                      ((sff[0] + sff[1]) + sff[2]) + sff[3]);
}

__global__ __launch_bounds__(256) void k_norm1(NormArgs g)
{
    if (!g.first && g.state->done) return;
    Idx<1> x{g.n, g.pitch, g.ppitch};
    double rr = 0.0, ff = 0.0;
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < g.n; p += gridDim.x * blockDim.x) {
        const double fv = g.f[p];
        const double r = fv - apply_pt<double, 1, false>(g.u, g.a, x, g.inv_h2, p + 1, 1, 1);
        rr += r * r;
        ff += fv * fv;
        if (g.r32) g.r32[p] = (float)r;
        if (g.r64) g.r64[p] = r;
    }
    norm_block_sum(rr, ff, g.partials, blockIdx.x);
}

// 2D: one wavefront takes B rows of 64 columns and marches down them.
// u, f and the coefficient are loaded once per point (the x neighbours are the
// adjacent lanes', the y neighbours the rows before and after; lanes 0 and 63
// also load the column beside the strip), and a face mean is computed once:
// the west face is the left lane's east face, the south face the previous
// row's north face.  Bandwidth bound for many systems; the thread-per-point
// form it replaces spent itself on four FP64 divisions and ten cache loads a
// point: 1023^2 diffusion 11.2 -> 9.9 us, 48 systems of 13.7 M unknowns
// 155 -> 88 us (all active).  A unit's loads are all in flight at once (four
// rows a round before: 2047^2 diffusion 24.8 -> 21.8 us, 4095^2 47.3 -> 44.8,
// 1023^2 diffusion 9.6 -> 9.4; 8 rows a unit).
// HASU false: the zero iterate (r = f), the same sums in the same order.
constexpr int kNormRows = 8;
// Rows a unit of a single system's norm takes: fewer where 8 give less than two
// wavefronts a SIMD (2048 units), which then wait on one unit's chain of loads and
// divisions.  A residual call, 8 / 2 / 1 rows and a thread a point: 255^2
// diffusion 21.8 / 19.9 / 19.6 / 19.4 us, 511^2 22.4 / 21.1 / 21.8 / 22.2, 1023^2
// 25.8 / 27.9 / 29.1 / 29.3.
static int norm2_rows(int n)
{
    const long long nsx = (n + 63) / 64;
    for (int b : {kNormRows, 2})
        if (nsx * ((n + b - 1) / b) >= 2048) return b;
    return 1;
}
template <bool VC, bool HASU, int B>
__device__ __forceinline__ void norm2_unit(const double *u, const double *f, const double *a, int n, long long pitch,
                                           double ih2, int ic, int j0, float *r32, double *r64, double &rr, double &ff)
{
    const int lane = threadIdx.x & 63;
    const int i = ic + lane;                                   // this lane's column
    const bool cin = i <= n;
    const int ie = lane == 0 ? ic - 1 : ic + 64;               // the column beside the strip (lanes 0, 63)
    const bool ein = (lane == 0 || lane == 63) && ie >= 1 && ie <= n;
    const int j1 = min(j0 + B, n + 1);
    auto row = [&](int j, double &c, double &e) {
        const bool ok = HASU && j >= 1 && j <= n;
        c = ok && cin ? gld(u + (long long)(j - 1) * pitch + (i - 1)) : 0.0;
        e = ok && ein ? gld(u + (long long)(j - 1) * pitch + (ie - 1)) : 0.0;
    };
    const int ia = min(i, n + 1), iae = min(ic + 64, n + 1);
    auto arow = [&](int j, double &c, double &e) {
        const long long o = (long long)min(j, n + 1) * (n + 2);
        c = gld(a + o + ia);
        e = lane == 63 ? gld(a + o + iae) : 0.0;
    };
    double us = 0.0, uc = 0.0, ue = 0.0, t = 0.0;  // the row before, the row, its side column
    row(j0 - 1, us, t);
    row(j0, uc, ue);
    double ac = 1.0, ae = 0.0, ws = 0.0;
    if constexpr (VC && HASU) {
        double as, ase;
        arow(j0 - 1, as, ase);
        arow(j0, ac, ae);
        ws = harm(as, ac);
    }
    double un[B], une[B], fv[B], an[B], ane[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
        row(j0 + k + 1, un[k], une[k]);
        fv[k] = cin && j0 + k <= n ? gld(f + (long long)(j0 + k - 1) * pitch + (i - 1)) : 0.0;
        if constexpr (VC && HASU) arow(j0 + k + 1, an[k], ane[k]);
    }
    // the strip's west faces of the rows, one a lane
    double wl = 0.0;
    if constexpr (VC && HASU) {
        const long long o = (long long)min(j0 + (lane & (B - 1)), n + 1) * (n + 2) + ic;
        wl = harm(gld(a + o - 1), gld(a + o));
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
        if (j0 + k >= j1) break;
        const double w = from_prev(uc, ue), e = from_next(uc, ue);
        double s = 0.0;
        if constexpr (!HASU) {
        } else if constexpr (!VC) {
            s = (uc - w) + (uc - e);
            s = (s + (uc - us)) + (uc - un[k]);
        } else {
            const double we = harm(ac, from_next(ac, ae)), ww = from_prev(we, lane_value(wl, k));
            const double wn = harm(ac, an[k]);
            s = ((ww * (uc - w) + we * (uc - e)) + ws * (uc - us)) + wn * (uc - un[k]);
            ws = wn;
            ac = an[k];
            ae = ane[k];
        }
        const double r = cin ? fv[k] - s * ih2 : 0.0;
        rr += r * r;
        ff += fv[k] * fv[k];
        // contiguous interior outputs
        const long long p = (long long)(j0 + k - 1) * n + (i - 1);
        if (cin && r32) gst(r32 + p, (float)r);
        if (cin && r64) gst(r64 + p, r);
        us = uc;
        uc = un[k];
        ue = une[k];
    }
}

template <bool VC, bool HASU, int B>
__global__ __launch_bounds__(256) void k_norm2(NormArgs g)
{
    if (!g.first && g.state->done) return;
    const int nsx = (g.n + 63) / 64, nunits = nsx * ((g.n + B - 1) / B);
    double rr = 0.0, ff = 0.0;
    for (int t = blockIdx.x * 4 + (threadIdx.x >> 6); t < nunits; t += gridDim.x * 4)
        norm2_unit<VC, HASU, B>(g.u, g.f, g.a, g.n, g.pitch, g.inv_h2, 1 + 64 * (t % nsx), 1 + B * (t / nsx), g.r32,
                                g.r64, rr, ff);
    norm_block_sum(rr, ff, g.partials, blockIdx.x);
}

// Work items of the batched norm: four strips of kNormRows rows of a system.
int norm_batch_items(int n) { return ((n + 255) / 256) * ((n + kNormRows - 1) / kNormRows); }
void norm_batch_item(int n, int q, NormItem &it)
{
    const int nx = (n + 255) / 256;
    it.i0 = 1 + 256 * (q % nx);
    it.j0 = 1 + kNormRows * (q / nx);
}
int norm2_blocks(int n)
{
    const int b = norm2_rows(n);
    const long long units = (long long)((n + 63) / 64) * ((n + b - 1) / b);
    return (int)std::min<long long>((units + 3) / 4, 2048);
}

// ---- 3D FP64 residual norm: each thread marches one column up a run of RUN
// planes keeping u(k - 1), u(k), u(k + 1) in registers, so every array is
// streamed once (the in-plane neighbours come from the cache); work units of
// 64 x 4 columns x RUN planes are dealt to the blocks in a fixed order.  8
// planes a unit up to 127 points an edge, where longer runs leave the chip
// waiting on a few columns (127^3 with the FP32 rhs written: 22.8 -> 13.4 us), 32
// above.  Those run with four wavefronts a SIMD: more of them push the rows that
// a neighbouring unit reads next out of the caches (511^3: 635 us with eight, 600
// with six, 569 with four; 255^3 72 / 69 / 66.5, and 74.5 in runs of 8).  The zero
// iterate reads f alone and keeps eight (511^3 212 us, 315 with four).
template <int RUN, bool HASU>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, RUN == 32 && HASU ? 4 : 8))) void k_norm3(NormArgs g)
{
    if (!g.first && g.state->done) return;
    Idx<3> x{g.n, g.pitch, g.ppitch};
    const int n = g.n;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int ntx = (n + 63) / 64, nty = (n + 3) / 4, ntz = (n + RUN - 1) / RUN;
    const long long nunits = (long long)ntx * nty * ntz;
    const double ih2 = g.inv_h2;
    const double *u = g.u;
    double rr = 0.0, ff = 0.0;
    auto U = [&](int i, int j, int k) -> double {
        return (HASU && i >= 1 && i <= n && j >= 1 && j <= n && k >= 1 && k <= n) ? u[x.off(i, j, k)] : 0.0;
    };
    for (long long un = blockIdx.x; un < nunits; un += gridDim.x) {
        const int i = (int)(un % ntx) * 64 + tx + 1, j = (int)((un / ntx) % nty) * 4 + ty + 1;
        const int k0 = (int)(un / ((long long)ntx * nty)) * RUN + 1, k1 = min(k0 + RUN, n + 1);
        if (i > n || j > n) continue;
        double dn = U(i, j, k0 - 1), c = U(i, j, k0);
#pragma unroll 4
        for (int k = k0; k < k1; ++k) {
            const double up = U(i, j, k + 1);
            const long long o = x.off(i, j, k);
            const double fv = g.f[o];
            double sa = (c - U(i - 1, j, k)) + (c - U(i + 1, j, k));
            sa = (sa + (c - U(i, j - 1, k))) + (c - U(i, j + 1, k));
            sa = (sa + (c - dn)) + (c - up);
            const double r = fv - sa * ih2;
            rr += r * r;
            ff += fv * fv;
            const long long pc = (long long)(i - 1) + (long long)n * ((j - 1) + (long long)n * (k - 1));
            if (g.r32) g.r32[pc] = (float)r;
            if (g.r64) g.r64[pc] = r;
            dn = c;
            c = up;
        }
    }
    norm_block_sum(rr, ff, g.partials, blockIdx.x);
}

// ---- batched FP64 residual (2D): a block per item, a wavefront per strip ------
__global__ __launch_bounds__(256) void k_norm_batch(const NormItem *items, const NormSys *sys, SolveState *states,
                                                    double *partials, int flags)
{
    const NormItem it = items[blockIdx.x];
    const NormSys S = sys[it.sys];
    if (!(flags & 1) && states[it.sys].done) return;
    double rr = 0.0, ff = 0.0;
    const int ic = it.i0 + 64 * (int)(threadIdx.x >> 6);
    float *r32 = (flags & 2) ? S.r32 : nullptr;
    if (ic <= S.n) {
        if (S.a) norm2_unit<true, true, kNormRows>(S.u, S.f, S.a, S.n, S.pitch, S.inv_h2, ic, it.j0, r32, nullptr, rr, ff);
        else norm2_unit<false, true, kNormRows>(S.u, S.f, S.a, S.n, S.pitch, S.inv_h2, ic, it.j0, r32, nullptr, rr, ff);
    }
    norm_block_sum(rr, ff, partials, it.slot);
}

hipError_t launch_norm_batch(const NormItem *items, int nitems, const NormSys *sys, SolveState *states,
                             double *partials, int flags, hipStream_t s)
{
    if (nitems <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_norm_batch, dim3(nitems), dim3(256), 0, s, items, sys, states, partials, flags);
    return hipGetLastError();
}

// The host may poll `done` while the stream runs on: one 8-byte store with nres,
// there when the kernel ends at the latest (its end makes all its stores visible
// to the host).  As an atomic store, of system or of device scope, a publishing
// kernel takes 4.6 us, 3.8 like this, three of them a solve: 255^2 287.6 -> 284.8.
__device__ __forceinline__ void publish_done(SolveState *pub, int done, int nres)
{
    static_assert(offsetof(SolveState, done) == 0 && offsetof(SolveState, nres) == 4, "one word");
    *reinterpret_cast<int2 *>(pub) = make_int2(done, nres);
}

// ---- reduction of the partial sums + stop test: one workgroup per system ----
// part0 / nparts: per-system slot ranges (device), or null for one system
// whose slots are [slot0, slot0 + nslots).
// A few hundred numbers: the launch and one round of loads.  Everything the
// kernel reads (partials, state, the whole history) is loaded at once, one
// value a thread; a single wavefront that walked the history in a loop took 4.5
// to 6.4 us of every cycle, this form 3.8 to 4.8.
__global__ __launch_bounds__(256) void k_norm_finish(SolveState *states, const double *partials, const int *part0,
                                                     const int *nparts, int slot0, int nslots, int first,
                                                     StateInit init, SolveState *pub)
{
    __shared__ double srr[4], sff[4], smn[4], shist[256];
    const int sys = blockIdx.x, tid = threadIdx.x;
    SolveState *st = states + sys;
    const int done0 = st->done, k = first ? 0 : st->nres, maxc = init.on ? init.maxc : st->maxc;
    const double tol = init.on ? init.tol : st->tol, watch = init.on ? init.watch : st->watch;
    const double stall = init.on ? init.stall : st->stall, ff0 = st->ff, rel0 = st->rel;
    const double h = tid <= 200 ? st->hist[tid] : 0.0;
    const int p0 = part0 ? part0[sys] : slot0;
    const int np = nparts ? nparts[sys] : nslots;
    double rr = 0.0, ff = 0.0;
    // four loads in flight per thread; thread t adds slots t, t + 256, ...
    for (int q0 = tid; q0 < np; q0 += 256 * 4) {
        double vr[4], vf[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = q0 + 256 * j;
            vr[j] = q < np ? partials[2 * (p0 + q)] : 0.0;
            vf[j] = q < np ? partials[2 * (p0 + q) + 1] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            rr += vr[j];
            ff += vf[j];
        }
    }
    if (!first && done0) {
        // stopped earlier: k residuals are recorded
        if (pub) {
            if (tid < k && tid <= 200) pub[sys].hist[tid] = h;
            if (tid == 0) {
                pub[sys].rel = rel0;
                publish_done(pub + sys, done0, k);
            }
        }
        return;
    }
    rr = wave_sum(rr);
    ff = wave_sum(ff);
    double mn = tid < k ? h : __builtin_inf();  // smallest of hist[0 .. k - 1]
    for (int o = 32; o > 0; o >>= 1) {
        const double x = __shfl_xor(mn, o, 64);
        mn = x < mn ? x : mn;
    }
    shist[tid] = h;
    if ((tid & 63) == 0) {
        srr[tid >> 6] = rr;
        sff[tid >> 6] = ff;
        smn[tid >> 6] = mn;
    }
    __syncthreads();
    if (pub && tid > 0 && tid <= k && tid <= 200) pub[sys].hist[tid - 1] = shist[tid - 1];
    if (tid != 0) return;
    rr = ((srr[0] + srr[1]) + srr[2]) + srr[3];
    ff = first ? ((sff[0] + sff[1]) + sff[2]) + sff[3] : ff0;
    for (int q = 1; q < 4; ++q) smn[0] = smn[q] < smn[0] ? smn[q] : smn[0];
    const double rel = sqrt(rr) / sqrt(ff);
    if (first) st->ff = ff;
    if (k <= 200) st->hist[k] = rel;
    st->rel = rel;
    st->nres = k + 1;
    int done = 0;
    if (!isfinite(rel)) done = 2;
    else if (rel <= tol) done = 1;
    else if (k >= 1 && watch > 0.0 && !(rel <= watch * shist[k - 1])) done = 4;
    else if (k <= 200) {
        const double last[4] = {rel, k >= 1 ? shist[k - 1] : 0.0, k >= 2 ? shist[k - 2] : 0.0,
                                k >= 3 ? shist[k - 3] : 0.0};
        const int rule = history_rule_of(last, k, rel < smn[0] ? rel : smn[0], stall);
        if (rule == 2) done = 6;
        else if (rule == 1) done = 5;
    }
    if (done == 0 && k >= maxc) done = 3;
    st->done = done;
    if (init.on) {
        st->maxc = maxc;
        st->tol = tol;
        st->watch = watch;
        st->stall = stall;
    }
    if (pub) {
        if (k <= 200) pub[sys].hist[k] = rel;
        pub[sys].rel = rel;
        publish_done(pub + sys, done, k + 1);
    }
}

hipError_t launch_norm_finish(SolveState *states, int nsys, const double *partials, const int *part0,
                              const int *nparts, int slot0, int nslots, int first, const StateInit &init,
                              SolveState *pub, hipStream_t s)
{
    hipLaunchKernelGGL(k_norm_finish, dim3(nsys), dim3(256), 0, s, states, partials, part0, nparts, slot0, nslots,
                       first, init, pub);
    return hipGetLastError();
}

// ---- FP64 correction u += e (state type S) -----------------------------------
template <class S>
__global__ __launch_bounds__(256) void k_ir_correct(double *u, long long pitch, long long ppitch, const S *e,
                                                    int n, int dim, SolveState *st)
{
    if (st && st->done) return;
    const long long m = npts(n, dim);
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(p, n, dim, i, j, k);
        const long long o = (long long)(i - 1) + (long long)(j - 1) * pitch + (long long)(k - 1) * ppitch;
        u[o] = u[o] + (double)Traits<S>::ld(e + p);
    }
}

// ---- setup: nodal coefficient hierarchy by injection ---------------------------
// Injection composes, so level l takes node (2^l I, 2^l J) of the finest array.
__global__ void k_coef_inject(const double *af, int nf, void *ac, int ncn, int stride, int as_float)
{
    const long long s = ncn + 2;
    const long long m = s * s;
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        const int I = (int)(p % s), J = (int)(p / s);
        const double v = af[(long long)stride * I + (long long)(nf + 2) * ((long long)stride * J)];
        if (as_float) ((float *)ac)[p] = (float)v;
        else ((double *)ac)[p] = v;
    }
}

__global__ void k_coef_check(const double *a, long long m, int *bad)
{
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        const double v = a[p];
        if (!(v > 0.0) || !isfinite(v)) atomicOr(bad, 1);
    }
}

// ---- s = D^-1 (f - A u) in FP64 (2D; a null = Poisson) --------------------------
__global__ __launch_bounds__(256) void k_scaled_residual64(const double *u, const double *f, const double *a, int n,
                                                           long long pitch, double *s)
{
    Idx<2> x{n, pitch, 0};
    const double ih2 = (double)(n + 1) * (n + 1);
    const long long m = (long long)n * n;
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < m; p += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(p % n) + 1, j = (int)(p / n) + 1;
        const long long o = x.off(i, j, 1);
        double r, dsum;
        if (a) {
            r = f[o] - apply_pt<double, 2, true>(u, a, x, ih2, i, j, 1);
            double ww, we, ws, wn;
            faces2d(a, n, i, j, ww, we, ws, wn);
            dsum = (((ww + we) + ws) + wn) * ih2;
        } else {
            r = f[o] - apply_pt<double, 2, false>(u, a, x, ih2, i, j, 1);
            dsum = 4.0 * ih2;
        }
        s[p] = r / dsum;
    }
}

hipError_t launch_scaled_residual64(const double *u, const double *f, const double *a, int n, long long pitch,
                                    double *s, hipStream_t st)
{
    const long long m = (long long)n * n;
    hipLaunchKernelGGL(k_scaled_residual64, dim3((int)std::min<long long>((m + 255) / 256, 65536)), dim3(256), 0, st,
                       u, f, a, n, pitch, s);
    return hipGetLastError();
}

// ---- launchers ---------------------------------------------------------------
static int grid_for(long long work, int block = 256)
{
    long long g = (work + block - 1) / block;
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    return (int)g;
}

template <class S, class F, bool VC>
static hipError_t rb_dim(const GenArgs &g, hipStream_t s)
{
    const long long half = (g.L.n + 1) / 2;
    const long long work = half * (g.L.dim > 1 ? g.L.n : 1) * (g.L.dim > 2 ? g.L.n : 1);
    const int grid = grid_for(work);
    switch (g.L.dim) {
    case 1: hipLaunchKernelGGL((k_rb_half<S, F, 1, false>), dim3(grid), dim3(256), 0, s, g); break;
    case 2: hipLaunchKernelGGL((k_rb_half<S, F, 2, VC>), dim3(grid), dim3(256), 0, s, g); break;
    case 3: hipLaunchKernelGGL((k_rb_half<S, F, 3, false>), dim3(grid), dim3(256), 0, s, g); break;
    }
    return hipGetLastError();
}

hipError_t launch_rb_half(int st, bool vc, const GenArgs &g, hipStream_t s)
{
    switch (st) {
    case ST_F64: return vc ? rb_dim<double, double, true>(g, s) : rb_dim<double, double, false>(g, s);
    case ST_F32: return vc ? rb_dim<float, float, true>(g, s) : rb_dim<float, float, false>(g, s);
    case ST_BF16: return vc ? rb_dim<bf16_t, float, true>(g, s) : rb_dim<bf16_t, float, false>(g, s);
    }
    return hipErrorInvalidValue;
}

template <class S, class F, bool VC>
static hipError_t jac_dim(const GenArgs &g, hipStream_t s)
{
    const int grid = grid_for(npts(g.L.n, g.L.dim));
    switch (g.L.dim) {
    case 1: hipLaunchKernelGGL((k_jacobi<S, F, 1, false>), dim3(grid), dim3(256), 0, s, g); break;
    case 2: hipLaunchKernelGGL((k_jacobi<S, F, 2, VC>), dim3(grid), dim3(256), 0, s, g); break;
    case 3: hipLaunchKernelGGL((k_jacobi<S, F, 3, false>), dim3(grid), dim3(256), 0, s, g); break;
    }
    return hipGetLastError();
}

hipError_t launch_jacobi(int st, bool vc, const GenArgs &g, hipStream_t s)
{
    switch (st) {
    case ST_F64: return vc ? jac_dim<double, double, true>(g, s) : jac_dim<double, double, false>(g, s);
    case ST_F32: return vc ? jac_dim<float, float, true>(g, s) : jac_dim<float, float, false>(g, s);
    case ST_BF16: return vc ? jac_dim<bf16_t, float, true>(g, s) : jac_dim<bf16_t, float, false>(g, s);
    }
    return hipErrorInvalidValue;
}

template <class S, class F, bool VC>
static hipError_t rr_dim(const GenArgs &g, hipStream_t s)
{
    const int grid = grid_for(npts(g.L.nc, g.L.dim));
    switch (g.L.dim) {
    case 1: hipLaunchKernelGGL((k_resid_restrict1<S, F>), dim3(grid), dim3(256), 0, s, g); break;
    case 2: {
        const long long units = (long long)((g.L.nc + 29) / 30) * ((g.L.nc + kRRows - 1) / kRRows);
        hipLaunchKernelGGL((k_resid_restrict2<S, F, VC>), dim3((unsigned)((units + 3) / 4)), dim3(256), 0, s, g);
        break;
    }
    case 3:
        hipLaunchKernelGGL((k_residual_to_a3<S, F>), dim3(grid_for(((long long)(g.L.n + 63) / 64) * ((g.L.n + 3) / 4) *
                                                               ((g.L.n + 31) / 32) * 256)),
                           dim3(256), 0, s, g);
        hipLaunchKernelGGL((k_restrict_from_a<S, F, 3>), dim3(grid), dim3(256), 0, s, g);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_resid_restrict(int st, bool vc, const GenArgs &g, hipStream_t s)
{
    switch (st) {
    case ST_F64: return vc ? rr_dim<double, double, true>(g, s) : rr_dim<double, double, false>(g, s);
    case ST_F32: return vc ? rr_dim<float, float, true>(g, s) : rr_dim<float, float, false>(g, s);
    case ST_BF16: return vc ? rr_dim<bf16_t, float, true>(g, s) : rr_dim<bf16_t, float, false>(g, s);
    }
    return hipErrorInvalidValue;
}

static unsigned pc2_grid(int n)
{
    const long long units = (long long)((n + 63) / 64) * ((n + 7) / 8);
    return (unsigned)((units + 3) / 4);
}

template <class S>
static hipError_t pc_dim(const GenArgs &g, hipStream_t s)
{
    const int grid = grid_for(npts(g.L.n, g.L.dim));
    switch (g.L.dim) {
    case 1: hipLaunchKernelGGL((k_prolong_correct1<S>), dim3(grid), dim3(256), 0, s, g); break;
    case 2: hipLaunchKernelGGL((k_prolong_correct2<S, true>), dim3(pc2_grid(g.L.n)), dim3(256), 0, s, g); break;
    case 3:
        hipLaunchKernelGGL((k_prolong_correct3<S>), dim3(grid_for(((long long)(g.L.n + 63) / 64) * ((g.L.n + 3) / 4) *
                                                                ((g.L.n + 31) / 32) * 256)),
                           dim3(256), 0, s, g);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_prolong_correct(int st, const GenArgs &g, hipStream_t s)
{
    switch (st) {
    case ST_F64: return pc_dim<double>(g, s);
    case ST_F32: return pc_dim<float>(g, s);
    case ST_BF16: return pc_dim<bf16_t>(g, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_restrict_rhs(int st, const GenArgs &g, hipStream_t s)
{
    const int grid = grid_for(npts(g.L.nc, g.L.dim));
#define MGX_RR(F)                                                                                   \
    switch (g.L.dim) {                                                                              \
    case 1: hipLaunchKernelGGL((k_restrict_rhs<F, 1>), dim3(grid), dim3(256), 0, s, g); break;      \
    case 2: hipLaunchKernelGGL((k_restrict_rhs<F, 2>), dim3(grid), dim3(256), 0, s, g); break;      \
    case 3: hipLaunchKernelGGL((k_restrict_rhs<F, 3>), dim3(grid), dim3(256), 0, s, g); break;      \
    }
    if (st == ST_F64) { MGX_RR(double) } else { MGX_RR(float) }
#undef MGX_RR
    return hipGetLastError();
}

hipError_t launch_interp(int st, const GenArgs &g, hipStream_t s)
{
    const int grid = grid_for(npts(g.L.n, g.L.dim));
#define MGX_IP(S)                                                                              \
    switch (g.L.dim) {                                                                         \
    case 1: hipLaunchKernelGGL((k_interp<S, 1>), dim3(grid), dim3(256), 0, s, g); break;       \
    case 2: hipLaunchKernelGGL((k_prolong_correct2<S, false>), dim3(pc2_grid(g.L.n)), dim3(256), 0, s, g); break; \
    case 3: hipLaunchKernelGGL((k_interp<S, 3>), dim3(grid), dim3(256), 0, s, g); break;       \
    }
    switch (st) {
    case ST_F64: MGX_IP(double) break;
    case ST_F32: MGX_IP(float) break;
    case ST_BF16: MGX_IP(bf16_t) break;
    }
#undef MGX_IP
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *p, long long bytes, hipStream_t s)
{
    const long long nw = bytes / 4;
    hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(nw)), dim3(256), 0, s, (uint32_t *)p, nw);
    return hipGetLastError();
}

hipError_t launch_zero_points(double *u, int n, int dim, long long pitch, long long ppitch, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_points, dim3(grid_for(npts(n, dim))), dim3(256), 0, s, u, n, dim, pitch, ppitch);
    return hipGetLastError();
}

hipError_t launch_copy_state(int st, const GenArgs &g, const void *src, void *dst, hipStream_t s)
{
    const int grid = grid_for(npts(g.L.n, g.L.dim));
#define MGX_COPY(S)                                                                                                   \
    switch (g.L.dim) {                                                                                                \
    case 1: hipLaunchKernelGGL((k_copy_state<S, 1>), dim3(grid), dim3(256), 0, s, g, (const S *)src, (S *)dst); break; \
    case 2: hipLaunchKernelGGL((k_copy_state<S, 2>), dim3(grid), dim3(256), 0, s, g, (const S *)src, (S *)dst); break; \
    case 3: hipLaunchKernelGGL((k_copy_state<S, 3>), dim3(grid), dim3(256), 0, s, g, (const S *)src, (S *)dst); break; \
    }
    switch (st) {
    case ST_F64: MGX_COPY(double) break;
    case ST_F32: MGX_COPY(float) break;
    case ST_BF16: MGX_COPY(bf16_t) break;
    }
#undef MGX_COPY
    return hipGetLastError();
}

template <int B>
static void launch_norm2(const NormArgs &a, int grid, hipStream_t s)
{
    if (!a.u) hipLaunchKernelGGL((k_norm2<false, false, B>), dim3(grid), dim3(256), 0, s, a);
    else if (a.a) hipLaunchKernelGGL((k_norm2<true, true, B>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_norm2<false, true, B>), dim3(grid), dim3(256), 0, s, a);
}

hipError_t launch_norm(const NormArgs &a, hipStream_t s)
{
    const int grid = a.nblocks;
    switch (a.dim) {
    case 1: hipLaunchKernelGGL(k_norm1, dim3(grid), dim3(256), 0, s, a); break;
    case 2:
        switch (norm2_rows(a.n)) {
        case 1: launch_norm2<1>(a, grid, s); break;
        case 2: launch_norm2<2>(a, grid, s); break;
        default: launch_norm2<kNormRows>(a, grid, s);
        }
        break;
    case 3:
        if (a.n <= 127) {
            if (a.u) hipLaunchKernelGGL((k_norm3<8, true>), dim3(grid), dim3(256), 0, s, a);
            else hipLaunchKernelGGL((k_norm3<8, false>), dim3(grid), dim3(256), 0, s, a);
        } else {
            if (a.u) hipLaunchKernelGGL((k_norm3<32, true>), dim3(grid), dim3(256), 0, s, a);
            else hipLaunchKernelGGL((k_norm3<32, false>), dim3(grid), dim3(256), 0, s, a);
        }
        break;
    }
    return hipGetLastError();
}

hipError_t launch_ir_correct(int st, double *u, long long pitch, long long ppitch, const void *e, int n, int dim,
                             SolveState *state, hipStream_t s)
{
    const int grid = grid_for(npts(n, dim));
    switch (st) {
    case ST_F64: hipLaunchKernelGGL((k_ir_correct<double>), dim3(grid), dim3(256), 0, s, u, pitch, ppitch, (const double *)e, n, dim, state); break;
    case ST_F32: hipLaunchKernelGGL((k_ir_correct<float>), dim3(grid), dim3(256), 0, s, u, pitch, ppitch, (const float *)e, n, dim, state); break;
    case ST_BF16: hipLaunchKernelGGL((k_ir_correct<bf16_t>), dim3(grid), dim3(256), 0, s, u, pitch, ppitch, (const bf16_t *)e, n, dim, state); break;
    }
    return hipGetLastError();
}

hipError_t launch_coef_inject(const double *af, int nf, void *ac, int ncn, int stride, int as_float, hipStream_t s)
{
    const long long m = (long long)(ncn + 2) * (ncn + 2);
    hipLaunchKernelGGL(k_coef_inject, dim3(grid_for(m)), dim3(256), 0, s, af, nf, ac, ncn, stride, as_float);
    return hipGetLastError();
}

hipError_t launch_coef_check(const double *a, long long count, int *bad, hipStream_t s)
{
    hipLaunchKernelGGL(k_coef_check, dim3(grid_for(count)), dim3(256), 0, s, a, count, bad);
    return hipGetLastError();
}

}  // namespace mgx
