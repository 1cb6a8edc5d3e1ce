// 1D red-black V-cycles in one wavefront, and whole 1D FP64 solves in one
// launch.
//
// The level of 2^K - 1 points gives each lane 2^(K - 6) consecutive points
// (the last lane's last point lies past the grid and stays zero), held with
// their right-hand side in registers; neighbours across lanes are DPP shifts by
// one lane, and a lane's even points are its points of the next coarser level.
// From 31 points down a level is packed onto the first lanes, one point each.
// No LDS arrays and no barriers: a half sweep is a few dozen instructions.
// What bounds it is the chain of about 100 such phases (ten levels, ten phases
// each); the level-by-level LDS form (k_tail.hip) paid an LDS round trip and a
// barrier of 16 wavefronts for each: an FP64 cycle of 1023 points takes 8.7 us
// from call to call, against 26.6 (2047: 11.5 against 31.5; 31: 8.0 against 13.3).
// W and F cycles repeat the visits of the levels below (solves of one cycle:
// 1023 FP64 W 1519 -> 221 us, 2047 F 190 -> 68, 1023 FP32 F 279 -> 77).  Full
// multigrid carries the rhs down first (solves with a full-multigrid start and
// no further cycle: 1023 169 -> 56 us, of F cycles 486 -> 98).
//
// k_solve1d keeps the solve in the registers too: the residual norm and the
// stop test follow each cycle in the wavefront (the other forms launch a norm
// and a stop-test kernel per cycle), so a solve is one launch: 1023 points FP64
// 71 -> 23 us (11.2 us of it the kernel), 2047 75 -> 26, 31 55 -> 17.
#include "dev_common.h"

namespace mgx {

namespace {

template <class S>
struct Tail1 {
    using T = Traits<S>;
    using C = typename T::C;
    int lane, nu1, nu2;
    double cinv;

    // points a lane holds on the level of 2^K - 1 points
    static constexpr int per(int K) { return K > 6 ? 1 << (K - 6) : 1; }

    // the point of (lane, s) is in the grid: s-th of m points a lane (0-based)
    template <int K>
    __device__ __forceinline__ bool in(int s) const
    {
        return per(K) * lane + s + 1 <= (1 << K) - 1;
    }

    template <int K>
    __device__ __forceinline__ void smooth(C (&u)[per(K)], const C (&f)[per(K)], int nsweeps)
    {
        constexpr int m = per(K);
        const C h2 = (C)(1.0 / (double)(1LL << (2 * K)));
        for (int sw = 0; sw < nsweeps; ++sw) {
            if constexpr (m == 1) {
#pragma unroll
                for (int colour = 0; colour < 2; ++colour) {
                    C s = h2 * f[0];
                    s = s + from_prev(u[0]);
                    s = s + from_next(u[0]);
                    const bool mine = ((lane + 1) & 1) == colour && in<K>(0);  // red: even 1-based index
                    u[0] = mine ? T::rnd(s * (C)0.5) : u[0];
                }
            } else {
                // red points (even index: odd s), then black ones
                const C right = from_next(u[0]);
#pragma unroll
                for (int s = 1; s < m; s += 2) {
                    C v = h2 * f[s];
                    v = v + u[s - 1];
                    v = v + (s + 1 < m ? u[s + 1 < m ? s + 1 : 0] : right);
                    u[s] = s + 1 < m || in<K>(s) ? T::rnd(v * (C)0.5) : (C)0;
                }
                const C left = from_prev(u[m - 1]);
#pragma unroll
                for (int s = 0; s < m; s += 2) {
                    C v = h2 * f[s];
                    v = v + (s > 0 ? u[s > 0 ? s - 1 : 0] : left);
                    v = v + u[s + 1];
                    u[s] = T::rnd(v * (C)0.5);
                }
            }
        }
    }

    template <int K>
    __device__ __forceinline__ void residual(const C (&u)[per(K)], const C (&f)[per(K)], C (&r)[per(K)])
    {
        constexpr int m = per(K);
        constexpr C ih2 = (C)(double)(1LL << (2 * K));
        const C left = from_prev(u[m - 1]), right = from_next(u[0]);
#pragma unroll
        for (int s = 0; s < m; ++s) {
            const C l = s > 0 ? u[s > 0 ? s - 1 : 0] : left, e = s + 1 < m ? u[s + 1 < m ? s + 1 : 0] : right;
            r[s] = in<K>(s) ? f[s] - ((u[s] - l) + (u[s] - e)) * ih2 : (C)0;
        }
    }

    // full weighting of a level's values onto the next coarser level
    template <int K>
    __device__ __forceinline__ void weight(const C (&r)[per(K)], C (&cf)[per(K - 1)])
    {
        constexpr int m = per(K), mc = per(K - 1);
        if constexpr (m > 1) {
            // coarse point s of the lane sits on its fine point 2 s + 1
            const C right = from_next(r[0]);
#pragma unroll
            for (int s = 0; s < mc; ++s) {
                C v = r[2 * s];
                v = v + (C)2 * r[2 * s + 1];
                v = v + (2 * s + 2 < m ? r[2 * s + 2 < m ? 2 * s + 2 : 0] : right);
                cf[s] = v * (C)0.25;
            }
            if (!in<K - 1>(mc - 1)) cf[mc - 1] = (C)0;
        } else {
            // one point a lane: coarse point I on fine point 2 I, packed to lane I - 1
            C v = from_prev(r[0]);
            v = v + (C)2 * r[0];
            v = v + from_next(r[0]);
            v = __shfl(v * (C)0.25, (2 * lane + 1) & 63, 64);
            cf[0] = lane < (1 << (K - 1)) - 1 ? v : (C)0;
        }
    }

    // u += the interpolation of the next coarser level's state
    template <int K>
    __device__ __forceinline__ void interpolate(const C (&cu)[per(K - 1)], C (&u)[per(K)])
    {
        constexpr int m = per(K), mc = per(K - 1);
        if constexpr (m > 1) {
            const C left = from_prev(cu[mc - 1]);
#pragma unroll
            for (int s = 0; s < mc; ++s) {
                const C l = s > 0 ? cu[s > 0 ? s - 1 : 0] : left;
                u[2 * s] = T::rnd(u[2 * s] + (l + cu[s]) * (C)0.5);
                u[2 * s + 1] = s + 1 < mc || in<K>(2 * s + 1) ? T::rnd(u[2 * s + 1] + cu[s]) : (C)0;
            }
        } else {
            constexpr int nc = (1 << (K - 1)) - 1;
            const int i = lane + 1, il = i >> 1, ir = (i + 1) >> 1;  // coarse indices left and right of i
            const C a = __shfl(cu[0], (il - 1) & 63, 64), b = __shfl(cu[0], (ir - 1) & 63, 64);
            const C cl = il >= 1 && il <= nc ? a : (C)0, cr = ir <= nc ? b : (C)0;
            const C corr = (i & 1) ? (cl + cr) * (C)0.5 : cl;
            u[0] = in<K>(0) ? T::rnd(u[0] + corr) : (C)0;
        }
    }

    // The visits of a level by one visit of its parent.
    template <int K, bool MULTI>
    __device__ __forceinline__ void below(C (&u)[per(K)], const C (&f)[per(K)], int kind)
    {
        if constexpr (MULTI && K > 1) {
            const int visits = visits_below(kind);
            for (int v = 0; v < visits; ++v) visit<K, true>(u, f, visit_kind(v, kind));
        } else {
            visit<K, MULTI>(u, f, kind);
        }
    }

    // One visit of the level of 2^K - 1 points, by a cycle of the given kind (V
    // unless MULTI).
    template <int K, bool MULTI>
    __device__ __forceinline__ void visit(C (&u)[per(K)], const C (&f)[per(K)], int kind)
    {
        if constexpr (K == 1) {
            // one unknown: FP64 inverse times rhs
            u[0] = lane == 0 ? T::rnd((C)(cinv * (double)f[0])) : (C)0;
        } else {
            constexpr int mc = per(K - 1);
            smooth<K>(u, f, nu1);
            C r[per(K)], cf[mc], cu[mc];
            residual<K>(u, f, r);
            weight<K>(r, cf);
#pragma unroll
            for (int s = 0; s < mc; ++s) cu[s] = (C)0;
            below<K - 1, MULTI>(cu, cf, kind);
            interpolate<K>(cu, u);
            smooth<K>(u, f, nu2);
        }
    }

    // Full multigrid from this level: f carried down by full weighting, the
    // coarsest level solved, then on each level the interpolated state and one
    // visit.
    template <int K>
    __device__ __forceinline__ void fmg(C (&u)[per(K)], const C (&f)[per(K)], int kind)
    {
        if constexpr (K == 1) {
            visit<1, true>(u, f, kind);
        } else {
            C cf[per(K - 1)], cu[per(K - 1)];
            weight<K>(f, cf);
            fmg<K - 1>(cu, cf, kind);
#pragma unroll
            for (int s = 0; s < per(K); ++s) u[s] = (C)0;
            interpolate<K>(cu, u);
            visit<K, true>(u, f, kind);
        }
    }
};

}  // namespace

// The tail of a 1D handle whose whole hierarchy is the tail: one cycle on the
// level L, or one full-multigrid pass.
template <class S, class F, int K, bool MULTI, bool FMG>
__global__ __launch_bounds__(64) void k_tail1d(TailArgs args, LevelDesc L)
{
    using T1 = Tail1<S>;
    using C = typename T1::C;
    constexpr int m = T1::per(K), n = (1 << K) - 1;
    const int lane = threadIdx.x;
    const int done = args.states[0].done;
    T1 t{lane, args.nu1, args.nu2, args.cinv[0]};
    C u[m], f[m];
#pragma unroll
    for (int s = 0; s < m; ++s) {
        const int i = m * lane + s;
        const bool ok = i < n;
        f[s] = ok ? (C)gld((const F *)L.f + i) : (C)0;
        u[s] = ok && !FMG && !L.uzero ? (C)Traits<S>::ld((const S *)L.B + i) : (C)0;
    }
    if (done) return;
    if constexpr (FMG) t.template fmg<K>(u, f, args.cycle);
    else t.template visit<K, MULTI>(u, f, args.cycle);
#pragma unroll
    for (int s = 0; s < m; ++s)
        if (m * lane + s < n) Traits<S>::st((S *)L.B + m * lane + s, u[s]);
}

// `cycles` V-cycles of the FP64 solve with the residual norm and the stop test
// after each; first: the solve's first norm in front of them (init sets the
// state), u read unless zero.  Stops with the state's done flag; pub: the
// host-visible copy of the state.
template <int K>
__global__ __launch_bounds__(64) void k_solve1d(double *u_, const double *f_, const double *cinv, int nu1, int nu2,
                                                SolveState *st, int first, int cycles, int zero, StateInit init,
                                                SolveState *pub)
{
    using T1 = Tail1<double>;
    constexpr int m = T1::per(K), n = (1 << K) - 1;
    const int lane = threadIdx.x;
    T1 t{lane, nu1, nu2, cinv[0]};
    double u[m], f[m];
#pragma unroll
    for (int s = 0; s < m; ++s) {
        const int i = m * lane + s;
        const bool ok = i < n;
        f[s] = ok ? gld(f_ + i) : 0.0;
        u[s] = ok && !zero ? gld(u_ + i) : 0.0;
    }
    // the state, in registers (the same in every lane)
    int done = first ? 0 : st->done, k = first ? 0 : st->nres;  // k: norms recorded
    const int maxc = first ? init.maxc : st->maxc;
    const double tol = first ? init.tol : st->tol;
    double ff = first ? 0.0 : st->ff, rel = first ? 0.0 : st->rel, smallest = __builtin_inf(), last[4] = {0, 0, 0, 0};
    for (int q = 0; q < k; ++q) smallest = fmin(smallest, st->hist[q]);
    for (int q = 0; q < 3 && q < k; ++q) last[q] = st->hist[k - 1 - q];
    auto norm = [&]() {
        double r[m], s = 0.0;
        t.template residual<K>(u, f, r);
#pragma unroll
        for (int q = 0; q < m; ++q) s += r[q] * r[q];
        if (k == 0) {
            double g = 0.0;
#pragma unroll
            for (int q = 0; q < m; ++q) g += f[q] * f[q];
            ff = wave_sum(g);
        }
        rel = sqrt(wave_sum(s)) / sqrt(ff);
        last[3] = last[2];
        last[2] = last[1];
        last[1] = last[0];
        last[0] = rel;
        smallest = rel < smallest ? rel : smallest;
        if (lane == 0 && k <= 200) {
            st->hist[k] = rel;
            pub->hist[k] = rel;
        }
        if (!isfinite(rel)) done = 2;
        else if (rel <= tol) done = 1;
        else if (k <= 200 && history_rule_of(last, k, smallest, 0.0) == 2) done = 6;
        if (done == 0 && k >= maxc) done = 3;
        ++k;
    };
    if (first) norm();
    for (int c = 0; c < cycles && !done; ++c) {
        t.template visit<K, false>(u, f, MG_CYCLE_V);
        norm();
    }
#pragma unroll
    for (int s = 0; s < m; ++s)
        if (m * lane + s < n) gst(u_ + m * lane + s, u[s]);
    if (lane == 0) {
        st->done = pub->done = done;
        st->nres = pub->nres = k;
        st->rel = pub->rel = rel;
        st->ff = ff;
        st->maxc = maxc;
        st->tol = tol;
        st->watch = st->stall = 0.0;
    }
}

// 32 points a lane (2047) fill the register file; 4095 would spill.  Below 31
// nothing is gained by a cycle of its own (the LDS form is launch bound there),
// but a solve is one launch instead of eight (7 points: 65 -> 20 us).
bool tail1d_supported(int n, int m) { return m == 1 && n >= 31 && n <= 2047; }
bool solve1d_supported(int n, int m) { return m == 1 && n <= 2047; }

#define MGX_T1_CASES(GO) \
    switch (n) {         \
    case 31: GO(5);      \
    case 63: GO(6);      \
    case 127: GO(7);     \
    case 255: GO(8);     \
    case 511: GO(9);     \
    case 1023: GO(10);   \
    case 2047: GO(11);   \
    }

template <class S, class F, bool MULTI, bool FMG>
static hipError_t tail1d_n(const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    const int n = L.n;
#define MGX_T1_GO(K)                                                                          \
    {                                                                                         \
        hipLaunchKernelGGL((k_tail1d<S, F, K, MULTI, FMG>), dim3(1), dim3(64), 0, s, a, L);   \
        return hipGetLastError();                                                             \
    }
    MGX_T1_CASES(MGX_T1_GO)
#undef MGX_T1_GO
    return hipErrorInvalidValue;
}
template <class S, class F>
static hipError_t tail1d_c(const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    return a.cycle != MG_CYCLE_V ? tail1d_n<S, F, true, false>(a, L, s) : tail1d_n<S, F, false, false>(a, L, s);
}

hipError_t launch_tail1d(int st, bool fmg, const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    if (a.nsys != 1) return hipErrorInvalidValue;
    switch (st) {
    case ST_F64: return fmg ? tail1d_n<double, double, true, true>(a, L, s) : tail1d_c<double, double>(a, L, s);
    case ST_F32: return tail1d_c<float, float>(a, L, s);
    case ST_BF16: return tail1d_c<bf16_t, float>(a, L, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_solve1d(int n, double *u, const double *f, const double *cinv, int nu1, int nu2, SolveState *st,
                          int first, int cycles, bool zero, const StateInit &init, SolveState *pub, hipStream_t s)
{
#define MGX_T1_GO(K)                                                                                              \
    {                                                                                                             \
        hipLaunchKernelGGL((k_solve1d<K>), dim3(1), dim3(64), 0, s, u, f, cinv, nu1, nu2, st, first, cycles,      \
                           zero ? 1 : 0, init, pub);                                                              \
        return hipGetLastError();                                                                                 \
    }
    switch (n) {
    case 1: MGX_T1_GO(1);
    case 3: MGX_T1_GO(2);
    case 7: MGX_T1_GO(3);
    case 15: MGX_T1_GO(4);
    }
    MGX_T1_CASES(MGX_T1_GO)
#undef MGX_T1_GO
    return hipErrorInvalidValue;
}

}  // namespace mgx
