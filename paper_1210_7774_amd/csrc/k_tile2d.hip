// LDS-tiled fused level kernels for the 2D levels of the cycle that do not
// fill the chip by marching.
//
// The row-marching kernels walk a chain of row steps (about a microsecond
// each) whose length is set by the block height plus the halo; on a level of
// a few hundred rows that chain, not the bytes, is the launch.  Here one
// workgroup owns a T x T tile and holds the tile plus a halo of R points in
// registers: every thread owns a pair of x-adjacent points, one of each colour
// (first column odd), with their right-hand side and face weights, for the
// whole launch.  Only the values of neighbours go through LDS, stored by
// colour class (all red points row by row, then all black ones), so the three
// neighbours a point does not own (its partner is in the thread) are reads of
// consecutive elements over a wavefront, without bank conflicts and without
// index arithmetic inside a stage.  A stage is one masked update, one LDS
// store and one barrier.  The halo shrinks by one ring per stage, so every
// value kept depends only on data the workgroup loaded itself (the fusion
// that the paper's blockable rule, "Vector Engine" section, forbids for
// elementwise kernels is legal through the recomputed halo).
//
// PRE  (mode 0): from u (or zero), nu red-black sweeps, residual, full
//   weighting onto the coarse points the tile owns; writes A and f_c.
// POST (mode 1): A + P u_c (bilinear), nu red-black sweeps; writes B, or adds
//   into the FP64 iterate (refinement), or also measures the squared residual
//   (the FP64 finest level).
//
// Tile edge (tile2d_edge): 32 points (28 for three sweeps, whose region would
// need more than 1024 threads), 16 where 32 would leave CUs idle: there the
// launch is load latency plus barriers, and 7 waves pass a barrier sooner than
// 16.  Measured (nu = 2, PRE / POST): 255 FP64 finest 15.4 / 16.6 us marching,
// 4.6 / 4.2 us here (T = 16); 511 FP64 8.4 / 8.8 us in the first tiled form (two
// strided passes over the region per stage, all values in LDS), 5.0 / 4.8 us
// here; 1023 FP64 18.8 / 20.7 -> 10.0 / 11.2 us; 1023 FP32 diffusion finest
// 36.1 / 49.8 us marching, 11.2 / 14.0 us here.  Where a launch has work for more
// than about three rounds of the chip marching is ahead (it recomputes one halo
// column in twelve instead of half the region): 2047 FP64 27 us a pass against 37.
#include "dev_common.h"

namespace mgx {

template <class C>
__device__ __forceinline__ C tharmonic(C a, C b)
{
    return (C)2 * a * b / (a + b);
}

// two x-adjacent values (aligned to one element)
template <class S>
__device__ __forceinline__ void ld2(const S *p, S &x, S &y)
{
    typedef S v2 __attribute__((ext_vector_type(2), aligned(sizeof(S))));
    const v2 v = *(const __attribute__((address_space(1))) v2 *)p;
    x = v.x;
    y = v.y;
}
template <class S>
__device__ __forceinline__ void st2(S *p, S x, S y)
{
    typedef S v2 __attribute__((ext_vector_type(2), aligned(sizeof(S))));
    *(__attribute__((address_space(1))) v2 *)p = (v2){x, y};
}
__device__ __forceinline__ double tval(double v) { return v; }
__device__ __forceinline__ float tval(float v) { return v; }
__device__ __forceinline__ float tval(bf16_t v) { return bf16_to_f32(v); }
__device__ __forceinline__ void tput(double &d, double v) { d = v; }
__device__ __forceinline__ void tput(float &d, float v) { d = v; }
// (values are rounded to bfloat16 when computed)
__device__ __forceinline__ void tput(bf16_t &d, float v) { d = (bf16_t)(__float_as_uint(v) >> 16); }

// FIN: the level may hold a system's finest level (POST: FP64 norm, or the add
// into the FP64 iterate).
template <class S, int MODE, int NS, int T, int FIN>
struct TileGeo {
    // halo: one ring per half sweep, and 2 more for residual + restriction, 1
    // (kept even: 2) for the norm
    static constexpr bool NORM = MODE == 1 && FIN && sizeof(S) == 8;
    static constexpr bool ACC = MODE == 1 && FIN && sizeof(S) < 8;
    static constexpr int R = 2 * NS + ((MODE == 0 || NORM) ? 2 : 0);
    static constexpr int LX = T + 2 * R, PX = LX / 2, NP = PX * LX;
    static constexpr int NT = (NP + 63) / 64 * 64;
};

template <class S, class F, bool VC, int MODE, int NS, int T, int FIN>
__global__ __launch_bounds__((TileGeo<S, MODE, NS, T, FIN>::NT)) void k_tile2d(MarchArgs args, LevelDesc L1)
{
    using G = TileGeo<S, MODE, NS, T, FIN>;
    using Tr = Traits<S>;
    using C = typename Tr::C;
    constexpr int R = G::R, LX = G::LX, PX = G::PX, NP = G::NP, NT = G::NT;
    static_assert(NT <= 1024 && R % 2 == 0 && T % 2 == 0, "tile geometry");
    __shared__ C U[2 * NP + 2];                            // red points, black points, a spare pair
    __shared__ C RP[MODE == 0 ? NP : 1], R0[MODE == 0 ? NP : 1];
    __shared__ C FE[VC ? NP : 1], FN0[VC ? NP : 1], FN1[VC ? NP : 1];
    __shared__ double wsum[G::NORM ? NT / 64 : 1];

    // Workgroups are dealt round-robin to the 8 XCDs; each gets a contiguous
    // range of tiles (neighbouring tiles' halos meet in one L2)
    const int per = (args.nitems + 7) / 8;
    const int item = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (item >= args.nitems) return;
    // items == null: one level, its descriptor in the arguments and its tiles
    // from the workgroup index (no dependent loads before the data)
    MarchItem wi;
    LevelDesc L;
    if (args.items == nullptr) {
        L = L1;
        const int tiles_x = (L.n + T - 1) / T;
        wi.ia = 1 + T * (item % tiles_x);
        wi.ja = 1 + T * (item / tiles_x);
        wi.part = item;
    } else {
        wi = uniform(args.items[item]);
        L = uniform(args.levels[wi.lvl]);
    }
    // the stop flag is tested once the region's loads are issued (the same
    // value for the whole workgroup)
    const int done = args.states[L.sys].done;
    const int n = L.n, nc = L.nc;
    const int tid = threadIdx.x;
    const bool act = NP == NT || tid < NP;
    const int y = act ? tid / PX : 0, kp = act ? tid % PX : 0;
    const int gi = wi.ia - R + 2 * kp, gj = wi.ja - R + y;  // the pair: columns gi (odd), gi + 1
    const bool rin = act && gj >= 1 && gj <= n && gi >= 1;
    const bool in0 = rin && gi <= n, in1 = rin && gi + 1 <= n;
    const C h2 = (C)L.h2, ih2 = (C)L.inv_h2;
    const int gic = min(max(gi, 1), n - 1), gjc = min(max(gj, 1), n);  // (n >= 3)
    const long long go = (long long)(gjc - 1) * L.pitch + (gic - 1);
    const bool edge = gi == n;                                         // the pair's first column is the last one
    const bool own = act && y >= R && y < R + T && kp >= R / 2 && kp < R / 2 + T / 2;

    // ---- load the region: clamped addresses, values selected afterwards, so
    // all of a thread's loads are in flight together
    const bool uzero = MODE == 0 && (L.uzero || args.zero_in);
    C ux[2] = {(C)0, (C)0}, fx[2];
    {
        F a, b;
        ld2((const F *)L.f + go, a, b);
        fx[0] = (C)(edge ? b : a);
        fx[1] = (C)b;
    }
    if (!uzero) {
        S a, b;
        ld2((const S *)(MODE == 0 ? L.B : L.A) + go, a, b);
        ux[0] = in0 ? tval(edge ? b : a) : (C)0;
        ux[1] = in1 ? tval(b) : (C)0;
    }
    double acc[2] = {0.0, 0.0};
    long long ao = 0;
    if constexpr (G::ACC) {
        ao = (long long)(gjc - 1) * L.acc_pitch + (gic - 1);
        if (L.acc && own && in0) {
            ld2(L.acc + ao, acc[0], acc[1]);
            if (edge) acc[0] = acc[1];
        }
    }
    C mid = (C)1, fe = (C)1, fn0 = (C)1, fn1 = (C)1;
    if constexpr (VC) {
        // the faces right of and above the pair's points (the boundary nodes
        // 0 and n + 1 have coefficients too); those left and below come from
        // the neighbours through LDS
        const C *ac = (const C *)L.a;
        auto node = [&](int i, int j) -> C {
            return gld(ac + (long long)min(max(j, 0), n + 1) * (n + 2) + min(max(i, 0), n + 1));
        };
        const C a0 = node(gi, gj), a1 = node(gi + 1, gj), a2 = node(gi + 2, gj);
        const C b0 = node(gi, gj + 1), b1 = node(gi + 1, gj + 1);
        mid = tharmonic(a0, a1);
        fe = tharmonic(a1, a2);
        fn0 = tharmonic(a0, b0);
        fn1 = tharmonic(a1, b1);
    }
    if constexpr (MODE == 1) {
        // bilinear coarse-grid correction: coarse (I, J) sits on fine (2I, 2J),
        // index 0 and nc + 1 are the zero boundary
        const S *bc = (const S *)L.Bc;
        const int I = (gi + 1) / 2;
        const int Ja = (gj & 1) ? (gj - 1) / 2 : gj / 2, Jb = (gj & 1) ? (gj + 1) / 2 : gj / 2;
        auto cv = [&](int i, int j) -> C {
            const bool ok = i >= 1 && i <= nc && j >= 1 && j <= nc;
            const C v = tval(gld(bc + (long long)(min(max(j, 1), nc) - 1) * L.cpitch + (min(max(i, 1), nc) - 1)));
            return ok ? v : (C)0;
        };
        const C l0 = cv(I - 1, Ja), r0 = cv(I, Ja), l1 = cv(I - 1, Jb), r1 = cv(I, Jb);
        const C x0a = (l0 + r0) * (C)0.5, x0b = (l1 + r1) * (C)0.5;
        const C c0 = (gj & 1) ? (x0a + x0b) * (C)0.5 : x0a;
        const C c1 = (gj & 1) ? (r0 + r1) * (C)0.5 : r0;
        ux[0] = in0 ? Tr::rnd(ux[0] + c0) : (C)0;
        ux[1] = in1 ? Tr::rnd(ux[1] + c1) : (C)0;
    }
    if (done) return;

    // ---- by colour class (0: red, 1-based index sum even) -----------------------
    const bool x1red = (gj & 1) == 0;  // which of the pair is red in this row
    const int q = y * PX + kp;
    const int dy = min(y, LX - 1 - y);
    const int dm0 = in0 ? min(min(2 * kp, LX - 1 - 2 * kp), dy) : -1;
    const int dm1 = in1 ? min(min(2 * kp + 1, LX - 2 - 2 * kp), dy) : -1;
    // distance of the class's point to the region's edge (stage test)
    const int dm[2] = {x1red ? dm1 : dm0, x1red ? dm0 : dm1};
    C u[2] = {x1red ? ux[1] : ux[0], x1red ? ux[0] : ux[1]};
    const C f[2] = {x1red ? fx[1] : fx[0], x1red ? fx[0] : fx[1]};
    int me[2], xn[2], yb[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        me[c] = act ? c * NP + q : 2 * NP + c;
        // the x neighbour that is not the partner: left of the first column,
        // right of the second (margins keep the clamped ones unused)
        const bool sec = (c == 0) == x1red;
        xn[c] = (1 - c) * NP + y * PX + min(max(kp + (sec ? 1 : -1), 0), PX - 1);
        yb[c] = (1 - c) * NP + min(max(y - 1, 0), LX - 3) * PX + kp;
    }
    // the point's west neighbour is its partner when it is the pair's second,
    // its east neighbour when it is the first (sums add west, east, south,
    // north: the order of the marching kernels, whose values these are)
    const bool second[2] = {x1red, !x1red};
    // face weights: west, east, south (row j - 1), north
    C fw[2], fE[2], fs[2], fn[2], id[2];
    if constexpr (VC) {
        if (act) {
            FE[q] = fe;
            FN0[q] = fn0;
            FN1[q] = fn1;
        }
        if (!uzero) {
            U[me[0]] = u[0];
            U[me[1]] = u[1];
        }
        __syncthreads();
        const C w = FE[max(q - 1, 0)], s0 = FN0[max(q - PX, 0)], s1 = FN1[max(q - PX, 0)];
        const C i0 = (C)1 / (((w + mid) + s0) + fn0), i1 = (C)1 / (((mid + fe) + s1) + fn1);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            fw[c] = second[c] ? mid : w;
            fE[c] = second[c] ? fe : mid;
            fs[c] = second[c] ? s1 : s0;
            fn[c] = second[c] ? fn1 : fn0;
            id[c] = second[c] ? i1 : i0;
        }
    }
    int m0 = 1;
    if (uzero) {
        // a zero state: the first red half sweep has no neighbours to read
        C v;
        if constexpr (VC) v = (h2 * f[0]) * id[0];
        else v = (h2 * f[0]) * (C)0.25;
        u[0] = dm[0] >= 1 ? Tr::rnd(v) : (C)0;
        m0 = 2;
    }
    if (!VC || uzero) {
        U[me[0]] = u[0];
        U[me[1]] = u[1];
        __syncthreads();
    }
    // ---- the red-black stages; stage m updates the points at least m from
    // the region's edge
#pragma unroll
    for (int m = 1; m <= 2 * NS; ++m) {
        if (m < m0) continue;
        const int c = (m & 1) ? 0 : 1;
        const C xo = U[xn[c]], up = U[yb[c]], dn = U[yb[c] + 2 * PX];
        const C w = second[c] ? u[1 - c] : xo, e = second[c] ? xo : u[1 - c];
        C v;
        if constexpr (!VC) v = ((((h2 * f[c] + w) + e) + up) + dn) * (C)0.25;
        else v = ((((h2 * f[c] + fw[c] * w) + fE[c] * e) + fs[c] * up) + fn[c] * dn) * id[c];
        if (dm[c] >= m) {
            u[c] = Tr::rnd(v);
            U[me[c]] = u[c];
        }
        if (m < 2 * NS || MODE == 0 || G::NORM) __syncthreads();
    }
    auto resid = [&](int c) -> C {
        const C xo = U[xn[c]], up = U[yb[c]], dn = U[yb[c] + 2 * PX];
        const C w = second[c] ? u[1 - c] : xo, e = second[c] ? xo : u[1 - c];
        C Au;
        if constexpr (!VC)
            Au = ((((u[c] - w) + (u[c] - e)) + (u[c] - up)) + (u[c] - dn)) * ih2;
        else
            Au = (((fw[c] * (u[c] - w) + fE[c] * (u[c] - e)) + fs[c] * (u[c] - up)) + fn[c] * (u[c] - dn)) * ih2;
        return f[c] - Au;
    };
    ux[0] = x1red ? u[1] : u[0];
    ux[1] = x1red ? u[0] : u[1];
    // ---- store the owned points
    if (own && in0) {
        if constexpr (G::ACC) {
            if (L.acc) {
                double *p = L.acc + ao;
                if (in1) st2(p, acc[0] + (double)ux[0], acc[1] + (double)ux[1]);
                else p[edge ? 1 : 0] = acc[0] + (double)ux[0];
            }
        }
        if (!G::ACC || !L.acc) {
            S *p = (S *)(MODE == 0 ? L.A : L.B) + go;
            S a, b;
            tput(a, ux[0]);
            tput(b, ux[1]);
            if (in1) st2(p, a, b);
            else gst(p + (edge ? 1 : 0), a);
        }
    }
    if constexpr (MODE == 0) {
        // ---- residual on the tile + 1, summed 1-2-1 along x, then along y
        const C rr[2] = {dm[0] >= R - 1 ? resid(0) : (C)0, dm[1] >= R - 1 ? resid(1) : (C)0};
        const C r0 = x1red ? rr[1] : rr[0], r1 = x1red ? rr[0] : rr[1];
        if (act) {
            RP[q] = r0 + (C)2 * r1;
            R0[q] = r0;
        }
        __syncthreads();
        // coarse (I, J) sits on fine (2I, 2J): the second point of a pair of an even row
        const int I = (gi + 1) / 2, J = gj / 2;
        if (own && in1 && (gj & 1) == 0 && I <= nc && J <= nc) {
            auto rx = [&](int p) { return RP[p] + R0[p + 1]; };
            const C v = ((rx(q - PX) + (C)2 * rx(q)) + rx(q + PX)) * (C)0.0625;
            gst((F *)L.fc + (long long)(J - 1) * L.cpitch + (I - 1), (F)v);
        }
    }
    if constexpr (G::NORM) {
        if (L.norm) {
            double s = 0.0;
            if (own) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const double r = dm[c] >= 0 ? (double)resid(c) : 0.0;
                    s += r * r;
                }
            }
            s = wave_sum(s);
            if ((tid & 63) == 0) wsum[tid >> 6] = s;
            __syncthreads();
            if (tid < 64) {
                double tot = 0.0;
                for (int k = 0; k < NT / 64; ++k) tot += wsum[k];
                put_partial(args.partials, wi.part, tot, 0.0);
            }
        }
    }
}

template <class S, class F, bool VC, int NS, int T>
static hipError_t tile_go(int mode, int fin, const MarchArgs &a, const LevelDesc &L, hipStream_t s)
{
    const dim3 grid((unsigned)((a.nitems + 7) / 8 * 8));
    if (mode == 0)
        hipLaunchKernelGGL((k_tile2d<S, F, VC, 0, NS, T, 0>), grid, dim3(TileGeo<S, 0, NS, T, 0>::NT), 0, s, a, L);
    else if (!fin)
        hipLaunchKernelGGL((k_tile2d<S, F, VC, 1, NS, T, 0>), grid, dim3(TileGeo<S, 1, NS, T, 0>::NT), 0, s, a, L);
    else
        hipLaunchKernelGGL((k_tile2d<S, F, VC, 1, NS, T, 1>), grid, dim3(TileGeo<S, 1, NS, T, 1>::NT), 0, s, a, L);
    return hipGetLastError();
}

template <class S, class F, bool VC>
static hipError_t tile_typed(int mode, int fin, int NS, const MarchArgs &a, const LevelDesc &L, hipStream_t s)
{
    const bool small = a.W == 16;
    switch (NS) {
    case 1: return small ? tile_go<S, F, VC, 1, 16>(mode, fin, a, L, s) : tile_go<S, F, VC, 1, 32>(mode, fin, a, L, s);
    case 2: return small ? tile_go<S, F, VC, 2, 16>(mode, fin, a, L, s) : tile_go<S, F, VC, 2, 32>(mode, fin, a, L, s);
    case 3: return small ? tile_go<S, F, VC, 3, 16>(mode, fin, a, L, s) : tile_go<S, F, VC, 3, 28>(mode, fin, a, L, s);
    }
    return hipErrorInvalidValue;
}

// tiles of count levels of n x n points: the large edge when that gives every
// one of the 256 CUs a tile, else 16
int tile2d_edge(int n, int count, int nsweeps)
{
    const int T = nsweeps == 3 ? 28 : 32, nt = (n + T - 1) / T;
    return (long long)nt * nt * count >= 256 ? T : 16;
}

hipError_t launch_tile2d(int mode, int st, bool vc, int nsweeps, bool finest, const MarchArgs &a, const LevelDesc &L,
                         hipStream_t s)
{
    if (a.nitems < 1 || a.W != a.Hb || (a.W != 16 && a.W != (nsweeps == 3 ? 28 : 32))) return hipErrorInvalidValue;
    const int fin = finest ? 1 : 0;
    switch (st) {
    case ST_F64: return vc ? tile_typed<double, double, true>(mode, fin, nsweeps, a, L, s)
                           : tile_typed<double, double, false>(mode, fin, nsweeps, a, L, s);
    case ST_F32: return vc ? tile_typed<float, float, true>(mode, fin, nsweeps, a, L, s)
                           : tile_typed<float, float, false>(mode, fin, nsweeps, a, L, s);
    default: return vc ? tile_typed<bf16_t, float, true>(mode, fin, nsweeps, a, L, s)
                       : tile_typed<bf16_t, float, false>(mode, fin, nsweeps, a, L, s);
    }
}

}  // namespace mgx
