// Coarse-level tail of the 3D red-black V-cycle (Poisson): one workgroup runs
// the levels of 15 and 7 points an edge and the 3^3 coarsest grid, each level's
// state and rhs in registers.
//
// As in the 2D tail, a level of 2^K - 1 points an edge is cut into 2 x 2 x 2
// blocks, one per thread (8^(K-1) of them; the last block along each axis
// reaches one point past the grid, which stays zero).  Point d of a block has
// the bits (x, y, z) of d set where its coordinate is even; its three
// neighbours inside the block are d with one bit flipped, and so is its
// neighbour outside along each axis, in the adjacent block (the one before for
// an odd coordinate, after for an even one).  Neighbours in x are the adjacent
// lane's (DPP), those in y and z go through LDS: four stores and eight loads a
// half sweep.  The 7-point level is one wavefront without workgroup barriers.
//
// Latency bound, about 25 dependent phases; the level-by-level LDS form
// (k_tail.hip) took 29.8 us (FP32) and 35.4 us (FP64) a cycle, this one 9.2 and
// 14.1 us.  W and F cycles repeat the visits of the levels below (solves of 7
// cycles: 63^3 FP32 W 1897 -> 810 us, FP64 F 1262 -> 813, 127^3 FP32 F 1879 -> 1477).
#include "dev_common.h"

namespace mgx {

namespace {

template <class C, int K>
struct T3Level {
    static constexpr int P = 1 << (K - 1);
    static constexpr int YS = P, ZS = (P + 2) * P, NB = (P + 2) * ZS;
    C v[8][NB];        // the eight points by block, a zero block row / plane on each side
    C r[6][NB];        // residuals of the points with an odd y or z (d < 6)
    C fc[P * P * P];
    C uc[(P + 1) * (P + 1) * (P + 1)];
};
template <class C, int K>
struct T3Lds {
    T3Level<C, K> top;
    T3Lds<C, K - 1> below;
};
template <class C>
struct T3Lds<C, 2> {};

template <class S>
struct Tail3 {
    using T = Traits<S>;
    using C = typename T::C;
    int tid, nu1, nu2;
    const double *cinv;  // LDS

    template <int K>
    static __device__ __forceinline__ bool active(int tid)
    {
        return tid < (1 << (3 * (K - 1)));
    }
    template <int K>
    static __device__ __forceinline__ void sync()
    {
        if constexpr (K >= 4) __syncthreads();
        else wave_sync();
    }

    // the neighbour of point d outside its block along each axis
    template <int K>
    static __device__ __forceinline__ void outer(const T3Level<C, K> &L, const C (&u)[8], int d, int q, C &x, C &y, C &z)
    {
        x = (d & 1) ? from_next(u[d ^ 1], (C)0) : from_prev(u[d ^ 1], (C)0);
        y = L.v[d ^ 2][(d & 2) ? q + L.YS : q - L.YS];
        z = L.v[d ^ 4][(d & 4) ? q + L.ZS : q - L.ZS];
    }

    template <int K>
    __device__ __forceinline__ void smooth(T3Level<C, K> &L, int nsweeps, C (&u)[8], const C (&f)[8], int q,
                                           const bool (&in)[8], bool last)
    {
        const C h2 = (C)(1.0 / (double)(1LL << (2 * K)));
        for (int sw = 0; sw < nsweeps; ++sw) {
#pragma unroll
            for (int colour = 0; colour < 2; ++colour) {
                if (active<K>(tid)) {
                    C v[8];
#pragma unroll
                    for (int d = 0; d < 8; ++d) {
                        // red: an even number of odd coordinates, i.e. an odd number of bits
                        if ((__builtin_popcount(d) & 1) == colour) continue;
                        C x, y, z;
                        outer<K>(L, u, d, q, x, y, z);
                        C s = h2 * f[d];
                        s = s + ((d & 1) ? u[d ^ 1] : x);
                        s = s + ((d & 1) ? x : u[d ^ 1]);
                        s = s + ((d & 2) ? u[d ^ 2] : y);
                        s = s + ((d & 2) ? y : u[d ^ 2]);
                        s = s + ((d & 4) ? u[d ^ 4] : z);
                        s = s + ((d & 4) ? z : u[d ^ 4]);
                        v[d] = in[d] ? T::rnd(s * (C)(1.0 / 6.0)) : (C)0;
                    }
#pragma unroll
                    for (int d = 0; d < 8; ++d) {
                        if ((__builtin_popcount(d) & 1) == colour) continue;
                        u[d] = v[d];
                        L.v[d][q] = v[d];
                    }
                }
                if (!(last && sw == nsweeps - 1 && colour == 1)) sync<K>();
            }
        }
    }

    // One visit of level K from the state u (its arrays are in LDS) with rhs f,
    // by a cycle of the given kind (V unless MULTI).
    template <int K, bool MULTI>
    __device__ __forceinline__ void visit(T3Lds<C, K> &lds, C (&u)[8], const C (&f)[8], bool last, int kind)
    {
        constexpr int P = 1 << (K - 1);
        constexpr C ih2 = (C)(double)(1LL << (2 * K));
        T3Level<C, K> &L = lds.top;
        const int px = tid % P, py = (tid / P) % P, pz = tid / (P * P);
        const int q = (pz + 1) * L.ZS + (py + 1) * L.YS + px;
        const bool ex = px < P - 1, ey = py < P - 1, ez = pz < P - 1;  // even coordinates in the grid
        bool in[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) in[d] = (ex || !(d & 1)) && (ey || !(d & 2)) && (ez || !(d & 4));
        smooth<K>(L, nu1, u, f, q, in, false);
        // ---- residual, full weighting onto the block's coarse point (its all-even point)
        C res[8];
        if (active<K>(tid)) {
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                C x, y, z;
                outer<K>(L, u, d, q, x, y, z);
                const C c = u[d];
                C s = (c - ((d & 1) ? u[d ^ 1] : x)) + (c - ((d & 1) ? x : u[d ^ 1]));
                s = (s + (c - ((d & 2) ? u[d ^ 2] : y))) + (c - ((d & 2) ? y : u[d ^ 2]));
                s = (s + (c - ((d & 4) ? u[d ^ 4] : z))) + (c - ((d & 4) ? z : u[d ^ 4]));
                res[d] = f[d] - s * ih2;
                if (d < 6) L.r[d][q] = res[d];
            }
        }
        sync<K>();
        if (active<K>(tid)) {
            C s = (C)0;
#pragma unroll
            for (int oz = 0; oz < 3; ++oz)
#pragma unroll
                for (int oy = 0; oy < 3; ++oy) {
                    // offsets -1, 0, +1: the block's odd, even coordinate, the next block's odd one
                    const int dyz = (oy == 1 ? 2 : 0) | (oz == 1 ? 4 : 0);
                    const int qq = q + (oy == 2 ? L.YS : 0) + (oz == 2 ? L.ZS : 0);
                    const bool own = oy != 2 && oz != 2;
                    const C r0 = own ? res[dyz] : L.r[dyz < 6 ? dyz : 0][qq];
                    const C r1 = own ? res[dyz | 1] : L.r[dyz < 6 ? dyz | 1 : 0][qq];
                    const int wyz = (oy == 1 ? 2 : 1) * (oz == 1 ? 2 : 1);
                    s = s + (C)wyz * r0;
                    s = s + (C)(2 * wyz) * r1;
                    s = s + (C)wyz * from_next(r0, (C)0);
                }
            L.fc[(pz * P + py) * P + px] = in[7] ? s * (C)0.015625 : (C)0;
        }
        sync<K>();
        // ---- the coarse level
        constexpr int U1 = P + 1;
        if constexpr (K == 3) {
            if (tid < 27) {
                double x = 0.0;
#pragma unroll
                for (int k = 0; k < 27; ++k)
                    x += cinv[tid * 27 + k] * (double)L.fc[((k / 9) * P + (k / 3) % 3) * P + k % 3];
                L.uc[((tid / 9 + 1) * U1 + (tid / 3) % 3 + 1) * U1 + tid % 3 + 1] = T::rnd((C)x);
            }
        } else if (tid < 64) {  // K == 4: the 7-point level in the first wavefront
            constexpr int Pc = P / 2;
            const int cx = tid % Pc, cy = (tid / Pc) % Pc, cz = tid / (Pc * Pc);
            C cf[8], cu[8];
            auto &B = lds.below.top;
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                cf[d] = L.fc[((2 * cz + (d >> 2)) * P + 2 * cy + ((d >> 1) & 1)) * P + 2 * cx + (d & 1)];
                cu[d] = (C)0;
                B.v[d][(cz + 1) * B.ZS + (cy + 1) * B.YS + cx] = (C)0;
            }
            wave_sync();
            if constexpr (MULTI) {
                const int visits = visits_below(kind);
                for (int v = 0; v < visits; ++v)
                    visit<K - 1, true>(lds.below, cu, cf, v == visits - 1, visit_kind(v, kind));
            } else {
                visit<K - 1, false>(lds.below, cu, cf, true, kind);
            }
#pragma unroll
            for (int d = 0; d < 8; ++d)
                L.uc[((2 * cz + 1 + (d >> 2)) * U1 + 2 * cy + 1 + ((d >> 1) & 1)) * U1 + 2 * cx + 1 + (d & 1)] = cu[d];
        }
        sync<K>();
        // ---- trilinear correction (x, then y, then z)
        if (active<K>(tid)) {
            const C *uc = L.uc + ((pz + 1) * U1 + py + 1) * U1 + px + 1;
            C pl[2][4];  // coarse plane K - 1 / K, by the (x, y) bits
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const C *b = uc - (1 - k) * U1 * U1;
                const C c11 = b[0], c01 = b[-1], c10 = b[-U1], c00 = b[-U1 - 1];
                const C l0 = (c00 + c10) * (C)0.5, l1 = (c01 + c11) * (C)0.5;
                pl[k][0] = (l0 + l1) * (C)0.5;
                pl[k][1] = (c10 + c11) * (C)0.5;
                pl[k][2] = l1;
                pl[k][3] = c11;
            }
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const C corr = (d & 4) ? pl[1][d & 3] : (pl[0][d & 3] + pl[1][d & 3]) * (C)0.5;
                u[d] = in[d] ? T::rnd(u[d] + corr) : (C)0;
                L.v[d][q] = u[d];
            }
        }
        sync<K>();
        smooth<K>(L, nu2, u, f, q, in, last);
    }
};

// zero the cells that are read before they are written (block arrays' borders,
// the coarse state's border)
template <class C, int K>
__device__ __forceinline__ void t3_zero(T3Lds<C, K> &lds, int tid, int nt)
{
    if constexpr (K > 2) {
        constexpr int P = 1 << (K - 1);
        using L = T3Level<C, K>;
        for (int q = tid; q < L::NB; q += nt) {
            const int y = (q / L::YS) % (P + 2), z = q / L::ZS;
            if (y >= 1 && y <= P && z >= 1 && z <= P) continue;
#pragma unroll
            for (int d = 0; d < 8; ++d) lds.top.v[d][q] = (C)0;
#pragma unroll
            for (int d = 0; d < 6; ++d) lds.top.r[d][q] = (C)0;
        }
        for (int q = tid; q < (P + 1) * (P + 1) * (P + 1); q += nt) lds.top.uc[q] = (C)0;
        t3_zero(lds.below, tid, nt);
    }
}

}  // namespace

template <class S, class F, int K, bool MULTI>
__global__ __launch_bounds__(K == 4 ? 512 : 64) void k_tail3d(TailArgs args, LevelDesc L)
{
    using T = Traits<S>;
    using C = typename T::C;
    constexpr int P = 1 << (K - 1), n = 2 * P - 1;
    __shared__ T3Lds<C, K> lds;
    __shared__ double cinv[27 * 27];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int done = args.states[0].done;
    const int px = tid % P, py = (tid / P) % P, pz = tid / (P * P);
    const int i = 2 * px + 1, j = 2 * py + 1, k = 2 * pz + 1;
    C u[8], f[8];
    long long o[8];
    bool in[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const int ii = i + (d & 1), jj = j + ((d >> 1) & 1), kk = k + (d >> 2);
        in[d] = ii <= n && jj <= n && kk <= n;
        o[d] = in[d] ? (long long)(ii - 1) + (long long)(jj - 1) * L.pitch + (long long)(kk - 1) * L.ppitch : 0;
        const C fv = (C)gld((const F *)L.f + o[d]);
        f[d] = in[d] ? fv : (C)0;
        u[d] = (C)0;
        if (!L.uzero) {
            const C uv = T::ld((const S *)L.B + o[d]);
            u[d] = in[d] ? uv : (C)0;
        }
    }
    for (int q = tid; q < 27 * 27; q += nt) cinv[q] = args.cinv[q];
    if (done) return;
    t3_zero(lds, tid, nt);
    using Lv = T3Level<C, K>;
#pragma unroll
    for (int d = 0; d < 8; ++d) lds.top.v[d][(pz + 1) * Lv::ZS + (py + 1) * Lv::YS + px] = u[d];
    __syncthreads();
    Tail3<S> t{tid, args.nu1, args.nu2, cinv};
    if constexpr (MULTI) {
        for (int v = 0; v < args.visits; ++v)
            t.template visit<K, true>(lds, u, f, v == args.visits - 1, visit_kind(v, args.cycle));
    } else {
        t.template visit<K, false>(lds, u, f, true, MG_CYCLE_V);
    }
    S *b = (S *)L.B;
#pragma unroll
    for (int d = 0; d < 8; ++d)
        if (in[d]) T::st(b + o[d], u[d]);
}

bool tail3d_supported(int n_top, int m) { return m == 27 && (n_top == 7 || n_top == 15); }

template <class S, class F, bool MULTI>
static hipError_t tail3d_k(const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    if (a.nsys != 1) return hipErrorInvalidValue;
    if (L.n == 15) hipLaunchKernelGGL((k_tail3d<S, F, 4, MULTI>), dim3(1), dim3(512), 0, s, a, L);
    else if (L.n == 7) hipLaunchKernelGGL((k_tail3d<S, F, 3, MULTI>), dim3(1), dim3(64), 0, s, a, L);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}
template <class S, class F>
static hipError_t tail3d_n(const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    return a.cycle != MG_CYCLE_V ? tail3d_k<S, F, true>(a, L, s) : tail3d_k<S, F, false>(a, L, s);
}

hipError_t launch_tail3d(int st, const TailArgs &a, const LevelDesc &L, hipStream_t s)
{
    switch (st) {
    case ST_F64: return tail3d_n<double, double>(a, L, s);
    case ST_F32: return tail3d_n<float, float>(a, L, s);
    case ST_BF16: return tail3d_n<bf16_t, float>(a, L, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace mgx
