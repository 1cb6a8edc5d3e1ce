// Coarse-level tail of the 2D red-black V-cycle: one workgroup per system
// runs every level from the tail's top level (63 points an edge or fewer) down
// to the 3 x 3 coarsest grid and back up, with each level's state, rhs and
// face weights in registers.
//
// A level of 2^K - 1 points an edge is cut into 2 x 2 blocks, one per thread
// (2^(K-1) x 2^(K-1) threads; the last column and row of blocks reach one
// point past the grid, which stays zero and doubles as the boundary).  A block
// holds two red points and two black ones, which are the four points' mutual
// neighbours; of the two neighbours a point has outside its block, the one in
// x is the adjacent lane's (DPP; the zero last column makes row ends right
// without masks) and the one in y goes through LDS, two stores and two loads a
// half sweep.  Blocks are also exactly the coarse points of the next level, so
// the restricted residual of block (p, r) is the rhs of coarse point (p, r).
// The levels of 15 points and fewer live in the first wavefront, which runs
// them without workgroup barriers.
//
// What bounds it is latency: about 45 dependent phases of one LDS round trip
// each.  The level-by-level LDS form (k_tail.hip, which keeps Jacobi and the
// sizes no register form covers) read every neighbour,
// the rhs and the faces from LDS with 16 wavefronts at a barrier per half sweep
// on every level: 29 us (63 .. 3, FP64) and 46 us (FP32 diffusion) against 11.8
// and 13.3 us here, of which about 2 us are the launch and 2 the first loads.
// Full multigrid with V-cycles on the tail's levels is the same kernel with
// the rhs carried down first: 72 us level by level, 23 us here (63 .. 3, FP64).
// W and F cycles repeat the visits of the levels below: solves with 6 cycles of
// 255^2 FP64 W 2455 -> 945 us, F 811 -> 512, of 63^2 FP32 diffusion F 732 -> 298
// (FP64 from 63 spills 54 registers there and is still the faster form).
#include "dev_common.h"

namespace mgx {

namespace {

// points of a block: the red ones, then the black ones
enum { RA = 0, RB = 1, BA = 2, BB = 3 };  // (odd, odd), (even, even), (even, odd), (odd, even) in (x, y)

// face weights of a block (diffusion): inside, and towards the eight outer neighbours
template <class C>
struct TFaces {
    C xo, xe, yo, ye;          // between the columns on the odd / even row, between the rows on the odd / even column
    C wo, we, eo, ee;          // west of (odd, odd), (odd, even); east of (even, odd), (even, even)
    C so, se, no, ne;          // south of (odd, odd), (even, odd); north of (odd, even), (even, even)
    C id[4];                   // 1 / sum of the faces, by point
};
template <class C>
struct TNone {};

template <class C>
__device__ __forceinline__ C t2harm(C a, C b)
{
    return (C)2 * a * b / (a + b);
}

// LDS of one level: the four points' arrays by block with a zero row above and
// below, two residual arrays likewise, the coarse rhs and the coarse state
// (with its zero border)
template <class C, int K>
struct TLevelLds {
    static constexpr int P = 1 << (K - 1);
    C v[4][(P + 2) * P];
    C r[2][(P + 2) * P];
    C fc[P * P];
    C uc[(P + 1) * (P + 1)];
};
template <class C, int K>
struct TLds {
    TLevelLds<C, K> top;
    TLds<C, K - 1> below;
};
template <class C>
struct TLds<C, 2> {};

template <class S, bool VC, int KTOP, bool MULTI>
struct Tail2 {
    using T = Traits<S>;
    using C = typename T::C;
    using FT = typename std::conditional<VC, TFaces<C>, TNone<C>>::type;

    int tid, nu1, nu2;
    const double *cinv;  // LDS
    FT faces[VC ? KTOP - 2 : 1];

    // blocks of level K sit on the first 4^(K-1) threads (all of them on the
    // top level, unless it is smaller than a wavefront)
    template <int K>
    static __device__ __forceinline__ bool active(int tid)
    {
        return (K == KTOP && K > 3) || tid < (1 << (2 * (K - 1)));
    }
    // levels of 15 points and fewer (K <= 4) fit in the first wavefront
    template <int K>
    static __device__ __forceinline__ void sync()
    {
        if constexpr (K >= 5) __syncthreads();
        else wave_sync();
    }

    template <int K>
    __device__ __forceinline__ void smooth(TLevelLds<C, K> &L, int nsweeps, C (&u)[4], const C (&f)[4], bool last)
    {
        constexpr int P = 1 << (K - 1);
        const C h2 = (C)(1.0 / (double)(1LL << (2 * K)));
        const int p = tid % P, r = tid / P, q = (r + 1) * P + p;
        const bool xin = p < P - 1, yin = r < P - 1;  // the even column / row is in the grid
        for (int sw = 0; sw < nsweeps; ++sw) {
            if (active<K>(tid)) {
                // red: the outer neighbours are black
                const C wA = from_prev(u[BA], (C)0), eB = from_next(u[BB], (C)0);
                const C sA = L.v[BB][q - P], nB = L.v[BA][q + P];
                C a, b;
                if constexpr (!VC) {
                    a = ((((h2 * f[RA] + wA) + u[BA]) + sA) + u[BB]) * (C)0.25;
                    b = ((((h2 * f[RB] + u[BB]) + eB) + u[BA]) + nB) * (C)0.25;
                } else {
                    const FT &w = faces[K - 3];
                    a = ((((h2 * f[RA] + w.wo * wA) + w.xo * u[BA]) + w.so * sA) + w.yo * u[BB]) * w.id[RA];
                    b = ((((h2 * f[RB] + w.xe * u[BB]) + w.ee * eB) + w.ye * u[BA]) + w.ne * nB) * w.id[RB];
                }
                u[RA] = T::rnd(a);
                u[RB] = (xin && yin) ? T::rnd(b) : (C)0;
                L.v[RA][q] = u[RA];
                L.v[RB][q] = u[RB];
            }
            sync<K>();
            if (active<K>(tid)) {
                const C eA = from_next(u[RA], (C)0), wB = from_prev(u[RB], (C)0);
                const C sA = L.v[RB][q - P], nB = L.v[RA][q + P];
                C a, b;
                if constexpr (!VC) {
                    a = ((((h2 * f[BA] + u[RA]) + eA) + sA) + u[RB]) * (C)0.25;
                    b = ((((h2 * f[BB] + wB) + u[RB]) + u[RA]) + nB) * (C)0.25;
                } else {
                    const FT &w = faces[K - 3];
                    a = ((((h2 * f[BA] + w.xo * u[RA]) + w.eo * eA) + w.se * sA) + w.ye * u[RB]) * w.id[BA];
                    b = ((((h2 * f[BB] + w.we * wB) + w.xe * u[RB]) + w.yo * u[RA]) + w.no * nB) * w.id[BB];
                }
                u[BA] = xin ? T::rnd(a) : (C)0;
                u[BB] = yin ? T::rnd(b) : (C)0;
                L.v[BA][q] = u[BA];
                L.v[BB][q] = u[BB];
            }
            if (!(last && sw == nsweeps - 1)) sync<K>();
        }
    }

    // Full weighting of a block's four values: coarse point (p, r) into L.fc.
    template <int K>
    __device__ __forceinline__ void weight(TLevelLds<C, K> &L, const C (&res)[4])
    {
        constexpr int P = 1 << (K - 1);
        const int p = tid % P, r = tid / P, q = (r + 1) * P + p;
        const bool xin = p < P - 1, yin = r < P - 1;
        if (active<K>(tid)) {
            L.r[0][q] = res[RA];
            L.r[1][q] = res[BA];
        }
        sync<K>();
        if (active<K>(tid)) {
            // rows 2r - 1, 2r, 2r + 1 of columns 2p - 1, 2p, 2p + 1, in order
            const C nRA = L.r[0][q + P], nBA = L.r[1][q + P];
            C s = res[RA];
            s = s + (C)2 * res[BA];
            s = s + from_next(res[RA], (C)0);
            s = s + (C)2 * res[BB];
            s = s + (C)4 * res[RB];
            s = s + (C)2 * from_next(res[BB], (C)0);
            s = s + nRA;
            s = s + (C)2 * nBA;
            s = s + from_next(nRA, (C)0);
            L.fc[r * P + p] = (xin && yin) ? s * (C)0.0625 : (C)0;
        }
        sync<K>();
    }

    // 3 x 3 unknowns: FP64 inverse times rhs
    __device__ __forceinline__ void coarsest(TLevelLds<C, 3> &L)
    {
        constexpr int P = 4;
        if (tid < 9) {
            double x = 0.0;
#pragma unroll
            for (int k = 0; k < 9; ++k) x += cinv[tid * 9 + k] * (double)L.fc[(k / 3) * P + k % 3];
            L.uc[(tid / 3 + 1) * (P + 1) + tid % 3 + 1] = T::rnd((C)x);
        }
    }

    // The next coarser level between a level's coarse rhs and its coarse
    // state: a V-cycle visit from zero, the visits of a W or F cycle (MULTI: two
    // W visits, or an F and then a V visit, the second from the first's
    // result), or full multigrid.
    template <int K, bool FMG>
    __device__ __forceinline__ void below(TLds<C, K> &lds, int kind)
    {
        constexpr int P = 1 << (K - 1), Pc = P / 2;
        TLevelLds<C, K> &L = lds.top;
        C cf[4], cu[4] = {(C)0, (C)0, (C)0, (C)0};
        const int pc = tid % Pc, rc = tid / Pc;
        if (active<K - 1>(tid)) {
            const C *fc = L.fc + 2 * rc * P + 2 * pc;
            cf[RA] = fc[0];
            cf[BA] = fc[1];
            cf[BB] = fc[P];
            cf[RB] = fc[P + 1];
            if constexpr (!FMG) {
                // the state starts from zero
#pragma unroll
                for (int k = 0; k < 4; ++k) lds.below.top.v[k][(rc + 1) * Pc + pc] = (C)0;
            }
        }
        sync<K - 1>();
        if constexpr (FMG) {
            fmg<K - 1>(lds.below, cu, cf, kind);
        } else if constexpr (MULTI) {
            const int visits = visits_below(kind);
            for (int v = 0; v < visits; ++v)
                visit<K - 1>(lds.below, cu, cf, v == visits - 1, visit_kind(v, kind));
        } else {
            visit<K - 1>(lds.below, cu, cf, true, kind);
        }
        if (active<K - 1>(tid)) {
            C *uc = L.uc + (2 * rc + 1) * (P + 1) + 2 * pc + 1;
            uc[0] = cu[RA];
            uc[1] = cu[BA];
            uc[P + 1] = cu[BB];
            uc[P + 2] = cu[RB];
        }
    }
    template <int K, bool FMG>
    __device__ __forceinline__ void coarse(TLds<C, K> &lds, int kind)
    {
        if constexpr (K == 3) {
            coarsest(lds.top);
        } else if constexpr (K == 5) {
            if (tid < 64) below<K, FMG>(lds, kind);  // the wavefront of the levels from here down
        } else {
            below<K, FMG>(lds, kind);
        }
        sync<K>();
    }

    // u (ADD: +=) the bilinear interpolation of the coarse state (coarse point
    // (p, r) is the block's (even, even) point)
    template <int K, bool ADD>
    __device__ __forceinline__ void interpolate(TLevelLds<C, K> &L, C (&u)[4])
    {
        constexpr int P = 1 << (K - 1);
        const int p = tid % P, r = tid / P, q = (r + 1) * P + p;
        const bool xin = p < P - 1, yin = r < P - 1;
        if (active<K>(tid)) {
            const C *uc = L.uc + (r + 1) * (P + 1) + p + 1;
            const C c11 = uc[0], c01 = uc[-1], c10 = uc[-(P + 1)], c00 = uc[-(P + 1) - 1];
            const C l0 = (c00 + c10) * (C)0.5, l1 = (c01 + c11) * (C)0.5;
            if constexpr (!ADD) u[0] = u[1] = u[2] = u[3] = (C)0;
            u[RA] = T::rnd(u[RA] + (l0 + l1) * (C)0.5);
            u[BA] = xin ? T::rnd(u[BA] + (c10 + c11) * (C)0.5) : (C)0;
            u[BB] = yin ? T::rnd(u[BB] + l1) : (C)0;
            u[RB] = (xin && yin) ? T::rnd(u[RB] + c11) : (C)0;
#pragma unroll
            for (int k = 0; k < 4; ++k) L.v[k][q] = u[k];
        }
        sync<K>();
    }

    // Full multigrid from level K with rhs f: f carried down by full weighting,
    // the coarsest level solved, then on each level the interpolated state and
    // one visit.
    template <int K>
    __device__ __forceinline__ void fmg(TLds<C, K> &lds, C (&u)[4], const C (&f)[4], int kind)
    {
        weight<K>(lds.top, f);
        coarse<K, true>(lds, kind);
        interpolate<K, false>(lds.top, u);
        visit<K>(lds, u, f, true, kind);
    }

    // One visit of level K from the state u (its four arrays are in LDS) with
    // rhs f, by a cycle of the given kind (V unless MULTI).
    template <int K>
    __device__ __forceinline__ void visit(TLds<C, K> &lds, C (&u)[4], const C (&f)[4], bool last, int kind)
    {
        constexpr int P = 1 << (K - 1);
        constexpr C ih2 = (C)(double)(1LL << (2 * K));
        TLevelLds<C, K> &L = lds.top;
        const int p = tid % P, r = tid / P, q = (r + 1) * P + p;
        const bool xin = p < P - 1, yin = r < P - 1;
        smooth<K>(L, nu1, u, f, false);
        // ---- residual, full weighting onto coarse point (p, r) of the block
        C res[4] = {(C)0, (C)0, (C)0, (C)0};
        if (active<K>(tid)) {
            const C w0 = from_prev(u[BA], (C)0), e1 = from_next(u[BB], (C)0);
            const C e2 = from_next(u[RA], (C)0), w3 = from_prev(u[RB], (C)0);
            const C s0 = L.v[BB][q - P], n1 = L.v[BA][q + P], s2 = L.v[RB][q - P], n3 = L.v[RA][q + P];
            C a[4];
            if constexpr (!VC) {
                a[RA] = ((u[RA] - w0) + (u[RA] - u[BA]) + (u[RA] - s0)) + (u[RA] - u[BB]);
                a[RB] = ((u[RB] - u[BB]) + (u[RB] - e1) + (u[RB] - u[BA])) + (u[RB] - n1);
                a[BA] = ((u[BA] - u[RA]) + (u[BA] - e2) + (u[BA] - s2)) + (u[BA] - u[RB]);
                a[BB] = ((u[BB] - w3) + (u[BB] - u[RB]) + (u[BB] - u[RA])) + (u[BB] - n3);
            } else {
                const FT &w = faces[K - 3];
                a[RA] = ((w.wo * (u[RA] - w0) + w.xo * (u[RA] - u[BA])) + w.so * (u[RA] - s0)) + w.yo * (u[RA] - u[BB]);
                a[RB] = ((w.xe * (u[RB] - u[BB]) + w.ee * (u[RB] - e1)) + w.ye * (u[RB] - u[BA])) + w.ne * (u[RB] - n1);
                a[BA] = ((w.xo * (u[BA] - u[RA]) + w.eo * (u[BA] - e2)) + w.se * (u[BA] - s2)) + w.ye * (u[BA] - u[RB]);
                a[BB] = ((w.we * (u[BB] - w3) + w.xe * (u[BB] - u[RB])) + w.yo * (u[BB] - u[RA])) + w.no * (u[BB] - n3);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) res[k] = f[k] - a[k] * ih2;
        }
        weight<K>(L, res);
        coarse<K, false>(lds, kind);
        interpolate<K, true>(L, u);
        smooth<K>(L, nu2, u, f, last);
    }

    // face weights of the block on level K from the nodal coefficient
    template <int K>
    __device__ __forceinline__ void load_faces(const C *a)
    {
        if constexpr (VC) {
            if (!active<K>(tid)) return;
            constexpr int P = 1 << (K - 1), n = 2 * P - 1, s = n + 2;
            const int i = 2 * (tid % P) + 1, j = 2 * (tid / P) + 1;  // the (odd, odd) point's node
            auto at = [&](int di, int dj) -> C { return gld(a + min(j + dj, n + 1) * s + min(i + di, n + 1)); };
            const C oo = at(0, 0), eo = at(1, 0), oe = at(0, 1), ee = at(1, 1);
            const C wo = at(-1, 0), we = at(-1, 1), xo = at(2, 0), xe = at(2, 1);
            const C so = at(0, -1), se = at(1, -1), no = at(0, 2), ne = at(1, 2);
            TFaces<C> &w = faces[K - 3];
            w.xo = t2harm(oo, eo);
            w.xe = t2harm(oe, ee);
            w.yo = t2harm(oo, oe);
            w.ye = t2harm(eo, ee);
            w.wo = t2harm(wo, oo);
            w.we = t2harm(we, oe);
            w.eo = t2harm(eo, xo);
            w.ee = t2harm(ee, xe);
            w.so = t2harm(so, oo);
            w.se = t2harm(se, eo);
            w.no = t2harm(oe, no);
            w.ne = t2harm(ee, ne);
            w.id[RA] = (C)1 / (((w.wo + w.xo) + w.so) + w.yo);
            w.id[BA] = (C)1 / (((w.xo + w.eo) + w.se) + w.ye);
            w.id[BB] = (C)1 / (((w.we + w.xe) + w.yo) + w.no);
            w.id[RB] = (C)1 / (((w.xe + w.ee) + w.ye) + w.ne);
        }
    }
};

// zero every LDS cell that is read before it is written: the rows above and
// below the blocks and the coarse state's border
template <class C, int K>
__device__ __forceinline__ void tail_zero(TLds<C, K> &lds, int tid, int nt)
{
    if constexpr (K > 2) {
        constexpr int P = 1 << (K - 1);
        for (int q = tid; q < P; q += nt) {
#pragma unroll
            for (int k = 0; k < 4; ++k) lds.top.v[k][q] = lds.top.v[k][(P + 1) * P + q] = (C)0;
            lds.top.r[0][(P + 1) * P + q] = lds.top.r[1][(P + 1) * P + q] = (C)0;
        }
        for (int q = tid; q < (P + 1) * (P + 1); q += nt) lds.top.uc[q] = (C)0;
        tail_zero(lds.below, tid, nt);
    }
}

}  // namespace

template <class S, class F, bool VC, int K, bool FMG, bool MULTI>
__global__ __launch_bounds__(K == 6 ? 1024 : K == 5 ? 256 : 64) void k_tail2d(TailArgs args, LevelDesc L1)
{
    using T = Traits<S>;
    using C = typename T::C;
    constexpr int P = 1 << (K - 1), n = 2 * P - 1;
    __shared__ TLds<C, K> lds;
    __shared__ double cinv[81];
    const int sys = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int done = args.states[sys].done;
    const LevelDesc *dl = args.levels + (long long)sys * args.nlev;
    // (a single system's top level comes in the arguments)
    const LevelDesc L = args.nsys == 1 ? L1 : dl[0];
    Tail2<S, VC, K, MULTI> t;
    t.tid = tid;
    t.nu1 = args.nu1;
    t.nu2 = args.nu2;
    t.cinv = cinv;
    const bool act = tid < P * P;
    const int p = tid % P, r = tid / P;
    const int i = 2 * p + 1, j = 2 * r + 1;
    const bool in[4] = {act, act && i < n && j < n, act && i < n, act && j < n};
    const int di[4] = {0, 1, 1, 0}, dj[4] = {0, 1, 0, 1};
    C u[4], f[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const long long o = in[k] ? (long long)(i - 1 + di[k]) + (long long)(j - 1 + dj[k]) * L.pitch : 0;
        const C fv = (C)gld((const F *)L.f + o);
        f[k] = in[k] ? fv : (C)0;
        u[k] = (C)0;
        if (!FMG && !L.uzero) {
            const C uv = T::ld((const S *)L.B + o);
            u[k] = in[k] ? uv : (C)0;
        }
    }
    for (int q = tid; q < 81; q += nt) cinv[q] = args.cinv[(long long)sys * 81 + q];
    if constexpr (VC) {
        // (the levels' coefficients: one descriptor each)
        t.template load_faces<K>((const C *)L.a);
        if constexpr (K > 3) t.template load_faces<K - 1>((const C *)dl[1].a);
        if constexpr (K > 4) t.template load_faces<K - 2>((const C *)dl[2].a);
        if constexpr (K > 5) t.template load_faces<K - 3>((const C *)dl[3].a);
    }
    if (done) return;
    tail_zero(lds, tid, nt);
    if (act) {
#pragma unroll
        for (int k = 0; k < 4; ++k) lds.top.v[k][(r + 1) * P + p] = u[k];
    }
    __syncthreads();
    if constexpr (FMG) {
        t.template fmg<K>(lds, u, f, args.cycle);
    } else if constexpr (MULTI) {
        for (int v = 0; v < args.visits; ++v)
            t.template visit<K>(lds, u, f, v == args.visits - 1, visit_kind(v, args.cycle));
    } else {
        t.template visit<K>(lds, u, f, true, MG_CYCLE_V);
    }
    S *b = (S *)L.B;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (in[k]) T::st(b + (long long)(i - 1 + di[k]) + (long long)(j - 1 + dj[k]) * L.pitch, u[k]);
}

template <class S, class F, bool VC, bool FMG, bool MULTI>
static hipError_t tail2d_n(const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    switch (L.n) {
    case 7: hipLaunchKernelGGL((k_tail2d<S, F, VC, 3, FMG, MULTI>), dim3(a.nsys), dim3(64), 0, s, a, L); break;
    case 15: hipLaunchKernelGGL((k_tail2d<S, F, VC, 4, FMG, MULTI>), dim3(a.nsys), dim3(64), 0, s, a, L); break;
    case 31: hipLaunchKernelGGL((k_tail2d<S, F, VC, 5, FMG, MULTI>), dim3(a.nsys), dim3(256), 0, s, a, L); break;
    case 63:
        // FP64 faces of four levels do not fit in the registers of 1024 threads
        if constexpr (!(VC && sizeof(S) == 8)) {
            hipLaunchKernelGGL((k_tail2d<S, F, VC, 6, FMG, MULTI>), dim3(a.nsys), dim3(1024), 0, s, a, L);
            break;
        }
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

bool tail2d_supported(int st, bool vc, int n_top, int m)
{
    if (m != 9) return false;
    if (n_top == 63) return !(vc && st == ST_F64);
    return n_top == 7 || n_top == 15 || n_top == 31;
}

template <class S, class F, bool FMG>
static hipError_t tail2d_s(bool vc, const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    if (a.cycle != MG_CYCLE_V)
        return vc ? tail2d_n<S, F, true, FMG, true>(a, L, s) : tail2d_n<S, F, false, FMG, true>(a, L, s);
    return vc ? tail2d_n<S, F, true, FMG, false>(a, L, s) : tail2d_n<S, F, false, FMG, false>(a, L, s);
}

hipError_t launch_tail2d(int st, bool vc, bool fmg, const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    switch (st) {
    case ST_F64: return fmg ? tail2d_s<double, double, true>(vc, a, L, s) : tail2d_s<double, double, false>(vc, a, L, s);
    case ST_F32: return tail2d_s<float, float, false>(vc, a, L, s);
    case ST_BF16: return tail2d_s<bf16_t, float, false>(vc, a, L, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace mgx
