// Pressure Poisson solve (paper Section 2.1: pressure equation of the fractional step,
// solved iteratively; multigrid and red-black Gauss-Seidel are among the solvers the paper
// evaluated) and the projection passes: divergence right-hand side, velocity correction,
// gauge.  Ghost equations (Section 2.2, Eq. 2) are refreshed after every fine-level sweep.
//
// Fine level (level 0) work is out of place between two pressure buffers; every pass reads
// one buffer and writes the other, so no pass ever reads a value another thread of the same
// pass writes.
#include <hip/hip_runtime.h>

#include <type_traits>

#include <cmath>
#include <utility>

#include "device_util.hpp"
#include "ibm_impl.hpp"
#include "zmarch.hpp"

namespace ibm {


// =======================================================================================
// ghost refresh: p_g = sum_{m != g} beta_m p_m + h_g from one snapshot (Jacobi over ghosts)
// fluid members are read from dst (already updated), ghost members from src_ghost (the
// values before this pass); degenerate ghosts take the mean of their fluid 26-neighbours.
// Weights are FP64; the right-hand sides gh may be absent (homogeneous error equation).
// =======================================================================================

// mean of p over a cell's fluid 26-neighbours (0 without any)
template <typename T>
__device__ inline double fluid_mean26(int64_t cell, int nx, int ny, int nz, const uint8_t *__restrict__ type,
                                      const T *p) {
    int i, j, k;
    unflatten(cell, nx, ny, i, j, k);
    double sm = 0.0;
    int n = 0;
    for (int dk = -1; dk <= 1; ++dk)
        for (int dj = -1; dj <= 1; ++dj)
            for (int di = -1; di <= 1; ++di) {
                const int ii = i + di, jj = j + dj, kk = k + dk;
                if (ii < 0 || jj < 0 || kk < 0 || ii >= nx || jj >= ny || kk >= nz) continue;
                const int64_t q = ((int64_t)kk * ny + jj) * nx + ii;
                if (type[q] == T_FLUID) {
                    sm += (double)p[q];
                    ++n;
                }
            }
    return n ? sm / n : 0.0;
}

// Eight lanes per ghost: lane m of a group takes stencil member m (the index and weight
// loads of a wave are contiguous and the eight gathers are in flight together), and the
// group sums its terms with three shuffle steps.  Degenerate ghosts (mean of the fluid
// 26-neighbours) are handled by the group's first lane.
constexpr int REFRESH_NT = 256;
// T: precision of the cycle (each new value is rounded to it); TS, TD: types of the two
// buffers (TD wider than T only after the widening last sweep of the mixed cycle).
template <typename T, typename TS = T, typename TD = T>
__global__ void __launch_bounds__(REFRESH_NT)
    k_ghost_refresh(GhostView G, const TS *__restrict__ src_ghost, TD *dst, int nx, int ny, int nz,
                    const uint8_t *__restrict__ type, const double *__restrict__ gh) {
    const int64_t g = ((int64_t)blockIdx.x * REFRESH_NT + threadIdx.x) >> 3;
    const int m = threadIdx.x & 7;
    const bool live = g < G.ng;
    const int64_t gc = live ? g : 0;
    const int32_t q = G.st[8 * gc + m];
    const double beta = G.beta[8 * gc + m];
    const unsigned gm = G.gmask[gc];
    const int32_t flags = G.flags[gc];
    // issued with the stencil loads, so the store needs no further round trip
    const int64_t cell = G.cell[gc];
    const double hg = gh ? gh[gc] : 0.0;
    double term = 0.0;
    if (live && q >= 0) term = beta * (double)(((gm >> m) & 1u) ? src_ghost[q] : dst[q]);
    term += __shfl_xor(term, 1, 64);
    term += __shfl_xor(term, 2, 64);
    term += __shfl_xor(term, 4, 64);
    if (!live || m != 0) return;
    double v;
    if (flags & GF_DEGENERATE) {
        v = fluid_mean26(cell, nx, ny, nz, type, dst);
    } else {
        v = gh ? term + hg : term;
    }
    dst[cell] = (TD)(T)v;
}

static GhostView ghost_view(ibm_grid *g) {
    GhostView G;
    G.ng = g->ng;
    G.cell = g->g_cell;
    G.st = g->g_st;
    G.gmask = g->g_mask;
    G.beta = g->g_beta;
    G.h = g->g_h;
    G.flags = g->g_flags;
    return G;
}

template <typename T>
static hipError_t launch_refresh(ibm_grid *g, const T *src_ghost, T *dst, const double *gh, hipStream_t s) {
    if (g->ng == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ghost_refresh<T>, dim3((unsigned)((8 * g->ng + REFRESH_NT - 1) / REFRESH_NT)),
                       dim3(REFRESH_NT), 0, s, ghost_view(g),
                       src_ghost, dst, g->nx, g->ny, g->nz, g->type, gh);
    return hipGetLastError();
}

// the refresh after the widening last sweep of the mixed cycle: FP32 arithmetic as in
// launch_refresh<float>, members read from the FP32 input and the FP64 result
static hipError_t launch_refresh_widen(ibm_grid *g, const float *src_ghost, double *dst, const double *gh,
                                       hipStream_t s) {
    if (g->ng == 0) return hipSuccess;
    hipLaunchKernelGGL((k_ghost_refresh<float, float, double>), dim3((unsigned)((8 * g->ng + REFRESH_NT - 1) / REFRESH_NT)),
                       dim3(REFRESH_NT), 0, s, ghost_view(g), src_ghost, dst, g->nx, g->ny, g->nz, g->type, gh);
    return hipGetLastError();
}

// =======================================================================================
// fine-level operator view helpers
// =======================================================================================

static Fine<double> fine64(ibm_grid *g) {
    Fine<double> F;
    F.nx = g->nx;
    F.ny = g->ny;
    F.nz = g->nz;
    F.axm = g->am0[0];
    F.axp = g->ap0[0];
    F.aym = g->am0[1];
    F.ayp = g->ap0[1];
    F.azm = g->am0[2];
    F.azp = g->ap0[2];
    F.wx = g->w0[0];
    F.wy = g->w0[1];
    F.wz = g->w0[2];
    F.type = g->type;
    F.inject = g->inject0;
    return F;
}
static Fine<float> fine32(ibm_grid *g) {
    Fine<float> F;
    F.nx = g->nx;
    F.ny = g->ny;
    F.nz = g->nz;
    F.axm = g->am0f[0];
    F.axp = g->ap0f[0];
    F.aym = g->am0f[1];
    F.ayp = g->ap0f[1];
    F.azm = g->am0f[2];
    F.azp = g->ap0f[2];
    F.wx = g->w0f[0];
    F.wy = g->w0f[1];
    F.wz = g->w0f[2];
    F.type = g->type;
    F.inject = g->inject0;
    return F;
}
template <typename T>
static Coarse<T> coarse_view(ibm_grid *g, int l);
template <>
Coarse<double> coarse_view<double>(ibm_grid *g, int l) {
    LevelHost &L = g->lev[l];
    Coarse<double> C;
    for (int d = 0; d < 3; ++d) {
        C.n[d] = L.n[d];
        C.w[d] = L.w64[d];
        C.Tl[d] = L.T64[d];
    }
    C.active = L.active;
    C.e = L.e64;
    C.R = L.R64;
    C.mu = &g->sc->mu[l];
    return C;
}
template <>
Coarse<float> coarse_view<float>(ibm_grid *g, int l) {
    LevelHost &L = g->lev[l];
    Coarse<float> C;
    for (int d = 0; d < 3; ++d) {
        C.n[d] = L.n[d];
        C.w[d] = L.w32[d];
        C.Tl[d] = L.T32[d];
    }
    C.active = L.active;
    C.e = L.e32;
    C.R = L.R32;
    C.mu = &g->sc->mu[l];
    return C;
}
static ProlongTab prolong_tab(ibm_grid *g, int l) {  // table of level l from level l+1
    ProlongTab P;
    for (int d = 0; d < 3; ++d) {
        P.lo[d] = g->lev[l].plo[d];
        P.hi[d] = g->lev[l].phi[d];
        P.t[d] = g->lev[l].pt[d];
        P.halved[d] = g->lev[l + 1].halved[d];
    }
    return P;
}

template <typename T>
static T *&level_e(LevelHost &L);
template <>
double *&level_e<double>(LevelHost &L) { return L.e64; }
template <>
float *&level_e<float>(LevelHost &L) { return L.e32; }
template <typename T>
static T *&level_e2(LevelHost &L);
template <>
double *&level_e2<double>(LevelHost &L) { return L.e64b; }
template <>
float *&level_e2<float>(LevelHost &L) { return L.e32b; }

template <typename T>
__device__ __forceinline__ void fine_stencil(const Fine<T> &F, const T *__restrict__ p, int i, int j, int k, int64_t id,
                                             T &num, T &diag) {
    const int64_t sy = F.nx, sz = (int64_t)F.nx * F.ny;
    const T axm = F.axm[i], axp = F.axp[i], aym = F.aym[j], ayp = F.ayp[j], azm = F.azm[k], azp = F.azp[k];
    T s = 0;
    s = s + (i > 0 ? axm * p[id - 1] : T(0));
    s = s + (i < F.nx - 1 ? axp * p[id + 1] : T(0));
    s = s + (j > 0 ? aym * p[id - sy] : T(0));
    s = s + (j < F.ny - 1 ? ayp * p[id + sy] : T(0));
    s = s + (k > 0 ? azm * p[id - sz] : T(0));
    s = s + (k < F.nz - 1 ? azp * p[id + sz] : T(0));
    T d = axm + axp;
    d = d + aym;
    d = d + ayp;
    d = d + azm;
    d = d + azp;
    num = s;
    diag = d;
}

template <typename T>
__device__ __forceinline__ void coarse_stencil(const Coarse<T> &L, const T *__restrict__ e, int I, int J, int K,
                                               int64_t id, T &num, T &diag) {
    const int64_t sy = L.n[0], sz = (int64_t)L.n[0] * L.n[1];
    const T txm = L.Tl[0][id], txp = (I < L.n[0] - 1) ? L.Tl[0][id + 1] : T(0);
    const T tym = L.Tl[1][id], typ = (J < L.n[1] - 1) ? L.Tl[1][id + sy] : T(0);
    const T tzm = L.Tl[2][id], tzp = (K < L.n[2] - 1) ? L.Tl[2][id + sz] : T(0);
    T s = 0;
    s = s + (I > 0 ? txm * e[id - 1] : T(0));
    s = s + (I < L.n[0] - 1 ? txp * e[id + 1] : T(0));
    s = s + (J > 0 ? tym * e[id - sy] : T(0));
    s = s + (J < L.n[1] - 1 ? typ * e[id + sy] : T(0));
    s = s + (K > 0 ? tzm * e[id - sz] : T(0));
    s = s + (K < L.n[2] - 1 ? tzp * e[id + sz] : T(0));
    T d = txm + txp;
    d = d + tym;
    d = d + typ;
    d = d + tzm;
    d = d + tzp;
    num = s;
    diag = d;
}

// =======================================================================================
// residual + restriction, fused with block partial sums of the coarse right-hand side
// =======================================================================================

// level l -> l+1 (l >= 1): R_{l+1}(C) = sum over active children of r, r = (R - V mu) - S e, for
// any child map, row-wise (the tiling of the level-0 restriction k_restrict0_map):
// a wave owns one coarse row J (one or two finer rows) of a window of coarse columns, a
// lane one finer column, and the lane marches up the finer planes with both rows in
// registers; the x neighbours and the high x face come from the adjacent lanes
// (the columns beside the window are loaded too), the high y face of the first row is the second
// row's low face, the high z face the next plane's low face, loaded with that plane.  Loads and
// lane moves as in the level-0 pass, for the same reason.  Per cell the operations
// are those of coarse_stencil; each lane sums its active cells over the rows and planes of
// the current coarse plane, and when that plane is complete lane I - I0 adds the sums of the
// one or two lanes holding the children of coarse column I.

template <typename T>
struct RCPlane {
    T en0, en1, tzn0, tzn1;  // e and the low z face of plane k+1
    T r0, r1, tx0, tx1, ty0, ty1;
    T ylo, yhi, tyh;         // e below the first and above the last row, the low y face above the last
    T w2;
    uint8_t a0, a1;
};

template <typename T, bool TWO, bool ONE>
__device__ __forceinline__ double resrestrict_row(const Coarse<T> &L, const Coarse<T> &C, const ChildMap &M, T mu,
                                                  const XTile &X, const XTile &Xe, int J, const ZTile &Z, int k1, int lane) {
    const int nx = L.n[0], ny = L.n[1], nz = L.n[2];
    const int64_t plane = (int64_t)nx * ny;
    const int I0 = X.I0, I1 = Xe.I0, fx0 = X.i0, fx1 = Xe.i0, k0 = Z.k0;
    const int i = fx0 - 1 + lane, zero = vector_zero();
    const bool inx = lane > 0 && i < fx1;
    const int ic = min(max(i, 0), nx - 1);
    const int ja = M.cs[1][J], jb = TWO ? ja + 1 : ja;
    const int64_t o0 = (int64_t)ja * nx + ic, o1 = (int64_t)jb * nx + ic;
    const int64_t olo = (int64_t)max(ja - 1, 0) * nx + ic, ohi = (int64_t)min(jb + 1, ny - 1) * nx + ic;
    const bool hx0 = ic > 0, hx1 = ic < nx - 1;
    const bool hy00 = ja > 0, hy10 = ja < ny - 1, hy01 = jb > 0, hy11 = jb < ny - 1;
    const T w0 = L.w[0][ic];
    const T vxy0 = w0 * L.w[1][ja], vxy1 = w0 * L.w[1][jb];
    const bool own = lane < I1 - I0;
    const int Io = min(I0 + lane, I1);
    const int ca = own ? M.cs[0][Io] - fx0 + 1 : 0;
    const bool pair = own && M.cs[0][min(Io + 1, I1)] - M.cs[0][Io] == 2;
    const int cb = min(ca + 1, 63);
    const T *__restrict__ pe = L.e;
    const T *__restrict__ pr = L.R;
    const T *__restrict__ px = L.Tl[0];
    const T *__restrict__ py = L.Tl[1];
    const T *__restrict__ pz = L.Tl[2];
    auto ld = [=](int k) -> RCPlane<T> {
        RCPlane<T> d;
        const int kk = min(k, nz - 1);
        const int64_t b = (int64_t)kk * plane, bn = (int64_t)min(kk + 1, nz - 1) * plane;
        d.en0 = pe[bn + o0];
        d.tzn0 = pz[bn + o0];
        d.r0 = pr[b + o0];
        d.tx0 = px[b + o0];
        d.ty0 = py[b + o0];
        d.a0 = L.active[b + o0];
        d.ylo = pe[b + olo];
        d.yhi = pe[b + ohi];
        d.tyh = py[b + ohi];
        if constexpr (TWO) {
            d.en1 = pe[bn + o1];
            d.tzn1 = pz[bn + o1];
            d.r1 = pr[b + o1];
            d.tx1 = px[b + o1];
            d.ty1 = py[b + o1];
            d.a1 = L.active[b + o1];
        } else {
            d.en1 = d.tzn1 = d.r1 = d.tx1 = d.ty1 = T(0);
            d.a1 = 0;
        }
        d.w2 = L.w[2][kk + zero];
        return d;
    };
    T em0 = (k0 > 0) ? pe[(int64_t)(k0 - 1) * plane + o0] : T(0);
    T ec0 = pe[(int64_t)k0 * plane + o0], tzc0 = pz[(int64_t)k0 * plane + o0];
    T em1 = T(0), ec1 = T(0), tzc1 = T(0);
    if constexpr (TWO) {
        em1 = (k0 > 0) ? pe[(int64_t)(k0 - 1) * plane + o1] : T(0);
        ec1 = pe[(int64_t)k0 * plane + o1];
        tzc1 = pz[(int64_t)k0 * plane + o1];
    }
    T acc = 0;
    double psum = 0.0;
    int K = Z.K0;
    // one cell of plane k: coarse_stencil's operations, then the residual
#define IBM_RC_CELL(TXM, TXP, TYM, TYP, TZM, TZP, XM, XP, YM, YP, ZM, ZP, EC, HY0, HY1, RV, VXY, W2, ACT)      \
    {                                                                                                          \
        const T txp_ = hx1 ? (TXP) : T(0), typ_ = (HY1) ? (TYP) : T(0), tzp_ = hz1_ ? (TZP) : T(0);            \
        T s_ = 0;                                                                                              \
        s_ = s_ + (hx0 ? (TXM) * (XM) : T(0));                                                                 \
        s_ = s_ + (hx1 ? txp_ * (XP) : T(0));                                                                  \
        s_ = s_ + ((HY0) ? (TYM) * (YM) : T(0));                                                               \
        s_ = s_ + ((HY1) ? typ_ * (YP) : T(0));                                                                \
        s_ = s_ + (hz0_ ? (TZM) * (ZM) : T(0));                                                                \
        s_ = s_ + (hz1_ ? tzp_ * (ZP) : T(0));                                                                 \
        T d_ = (TXM) + txp_;                                                                                   \
        d_ = d_ + (TYM);                                                                                       \
        d_ = d_ + typ_;                                                                                        \
        d_ = d_ + (TZM);                                                                                       \
        d_ = d_ + tzp_;                                                                                        \
        const T vol_ = (VXY) * (W2);                                                                           \
        const T rc_ = ((RV) - vol_ * mu) - (s_ - d_ * (EC));                                                   \
        acc += (in_ && (ACT)) ? rc_ : T(0);                                                                    \
    }
#define IBM_RC_PLANE(D, kk)                                                                                    \
    {                                                                                                          \
        const int k_ = (kk);                                                                                   \
        const bool hz0_ = k_ > 0, hz1_ = k_ < nz - 1, in_ = inx && k_ < k1;                                    \
        /* in every lane, not inside the selections below */                                                   \
        const T su0_ = lane_below(ec0), sd0_ = lane_above(ec0), st0_ = lane_above((D).tx0);                    \
        IBM_RC_CELL((D).tx0, st0_, (D).ty0, TWO ? (D).ty1 : (D).tyh, tzc0, (D).tzn0, su0_, sd0_, (D).ylo,      \
                    TWO ? ec1 : (D).yhi, em0, (D).en0, ec0, hy00, hy10, (D).r0, vxy0, (D).w2, (D).a0 != 0);    \
        if constexpr (TWO) {                                                                                   \
            const T su1_ = lane_below(ec1), sd1_ = lane_above(ec1), st1_ = lane_above((D).tx1);                \
            IBM_RC_CELL((D).tx1, st1_, (D).ty1, (D).tyh, tzc1, (D).tzn1, su1_, sd1_, ec0, (D).yhi, em1,        \
                        (D).en1, ec1, hy01, hy11, (D).r1, vxy1, (D).w2, (D).a1 != 0);                          \
        }                                                                                                      \
        if ((Z.ends >> (k_ - k0)) & 1) { /* the coarse plane K is complete */                                   \
            T s = __shfl(acc, ca, 64);                                                                         \
            const T s2 = __shfl(acc, cb, 64);                                                                  \
            if (pair) s = s + s2;                                                                              \
            if (own) {                                                                                         \
                const int64_t cid = ((int64_t)K * C.n[1] + J) * C.n[0] + I0 + lane;                            \
                C.R[cid] = s;                                                                                  \
                if (C.e) C.e[cid] = T(0);                                                                      \
                psum += (double)s;                                                                             \
            }                                                                                                  \
            acc = T(0);                                                                                        \
            ++K;                                                                                               \
        }                                                                                                      \
        em0 = ec0;                                                                                             \
        ec0 = (D).en0;                                                                                         \
        tzc0 = (D).tzn0;                                                                                       \
        em1 = ec1;                                                                                             \
        ec1 = (D).en1;                                                                                         \
        tzc1 = (D).tzn1;                                                                                       \
    }
    RCPlane<T> qa = ld(k0);
    if constexpr (ONE) {  // a level of one plane
        IBM_RC_PLANE(qa, k0);
        return psum;
    }
    RCPlane<T> qb;
    for (int k = k0; k < k1; k += 2) {  // no way out in between, as in the level-0 pass
        qb = ld(k + 1);
        IBM_RC_PLANE(qa, k);
        qa = ld(k + 2);
        IBM_RC_PLANE(qb, k + 1);
    }
#undef IBM_RC_PLANE
#undef IBM_RC_CELL
    return psum;
}

template <typename T, bool ONE>
__global__ void __launch_bounds__(RM_NT)
    k_resrestrictC_map(Coarse<T> L, Coarse<T> C, ChildMap M, RowTiles t, double *partials) {
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const T mu = (T)(*L.mu);
    double psum = 0.0;
    const int per = gridDim.x >> 3;  // the grid is a multiple of 8
    for (int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3); tile < t.ntiles; tile += gridDim.x) {
        int q = tile;
        const int txi = q % t.ntx;
        q /= t.ntx;
        const int tyi = q % t.nty;
        const int chunk = q / t.nty;
        const int J = tyi * RM_W + wave;
        const XTile X = M.tx[txi], Xe = M.tx[txi + 1];
        const ZTile Z = M.tz[chunk];
        const int k1 = M.tz[chunk + 1].k0;
        if (J >= C.n[1] || X.I0 >= Xe.I0 || Z.k0 >= k1) continue;
        if (M.cs[1][J + 1] - M.cs[1][J] == 2)
            psum += resrestrict_row<T, true, ONE>(L, C, M, mu, X, Xe, J, Z, k1, lane);
        else
            psum += resrestrict_row<T, false, ONE>(L, C, M, mu, X, Xe, J, Z, k1, lane);
    }
    __shared__ double sh[RM_NT / 64];
    const double tot = block_sum<RM_NT>(psum, sh, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// The same for a level pair with every axis halved: a thread per coarse cell loads its
// 2 x 2 x 2 children as x pairs (one vector access per row and array), the neighbour layers
// around the block and the high-face transmissibilities once, all before any arithmetic,
// instead of rebuilding each child's stencil from scalar loads.  Per child the operations
// are those of coarse_stencil, and the children are summed in the same order (x fastest,
// then y, then z).
template <typename T>
__global__ void __launch_bounds__(256) k_resrestrictC8(Coarse<T> L, Coarse<T> C, double *partials) {
    using V = typename Pair2<T>::type;
    __shared__ double sh[4];
    const int64_t NC = (int64_t)C.n[0] * C.n[1] * C.n[2];
    const int64_t cid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double Rsum = 0.0;
    if (cid < NC) {
        int I, J, K;
        unflatten(cid, C.n[0], C.n[1], I, J, K);
        const int n0 = L.n[0], n1 = L.n[1], n2 = L.n[2];
        const int64_t sy = n0, sz = (int64_t)n0 * n1;
        const int i0 = 2 * I, j0 = 2 * J, k0 = 2 * K;
        const int im = max(i0 - 1, 0), ip = min(i0 + 2, n0 - 1);
        const int jm = max(j0 - 1, 0), jp = min(j0 + 2, n1 - 1);
        const int km = max(k0 - 1, 0), kp = min(k0 + 2, n2 - 1);
        auto at = [&](int j, int k) -> int64_t { return (int64_t)k * sz + (int64_t)j * sy; };
        V E[2][2], RR[2][2], X[2][2], Y[2][2], Z[2][2];
        T Exm[2][2], Exp[2][2], Xh[2][2];
        uint16_t A[2][2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int64_t r = at(j0 + b, k0 + c);
                E[b][c] = *reinterpret_cast<const V *>(L.e + r + i0);
                RR[b][c] = *reinterpret_cast<const V *>(L.R + r + i0);
                X[b][c] = *reinterpret_cast<const V *>(L.Tl[0] + r + i0);
                Y[b][c] = *reinterpret_cast<const V *>(L.Tl[1] + r + i0);
                Z[b][c] = *reinterpret_cast<const V *>(L.Tl[2] + r + i0);
                A[b][c] = *reinterpret_cast<const uint16_t *>(L.active + r + i0);
                Exm[b][c] = L.e[r + im];
                Exp[b][c] = L.e[r + ip];
                Xh[b][c] = L.Tl[0][r + ip];
            }
        V EYm[2], EYp[2], YH[2], EZm[2], EZp[2], ZH[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            EYm[q] = *reinterpret_cast<const V *>(L.e + at(jm, k0 + q) + i0);
            EYp[q] = *reinterpret_cast<const V *>(L.e + at(jp, k0 + q) + i0);
            YH[q] = *reinterpret_cast<const V *>(L.Tl[1] + at(jp, k0 + q) + i0);
            EZm[q] = *reinterpret_cast<const V *>(L.e + at(j0 + q, km) + i0);
            EZp[q] = *reinterpret_cast<const V *>(L.e + at(j0 + q, kp) + i0);
            ZH[q] = *reinterpret_cast<const V *>(L.Tl[2] + at(j0 + q, kp) + i0);
        }
        const T mu = (T)(*L.mu);
        T R = 0;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const int i = i0 + a, j = j0 + b, k = k0 + c;
                    const T ev = a ? E[b][c].y : E[b][c].x;
                    const T txm = a ? X[b][c].y : X[b][c].x;
                    const T txp = a ? ((i < n0 - 1) ? Xh[b][c] : T(0)) : X[b][c].y;
                    const T tym = a ? Y[b][c].y : Y[b][c].x;
                    const T typ = b ? ((j < n1 - 1) ? (a ? YH[c].y : YH[c].x) : T(0)) : (a ? Y[1][c].y : Y[1][c].x);
                    const T tzm = a ? Z[b][c].y : Z[b][c].x;
                    const T tzp = c ? ((k < n2 - 1) ? (a ? ZH[b].y : ZH[b].x) : T(0)) : (a ? Z[b][1].y : Z[b][1].x);
                    const T exm = a ? E[b][c].x : Exm[b][c];
                    const T exp = a ? Exp[b][c] : E[b][c].y;
                    const T eym = b ? (a ? E[0][c].y : E[0][c].x) : (a ? EYm[c].y : EYm[c].x);
                    const T eyp = b ? (a ? EYp[c].y : EYp[c].x) : (a ? E[1][c].y : E[1][c].x);
                    const T ezm = c ? (a ? E[b][0].y : E[b][0].x) : (a ? EZm[b].y : EZm[b].x);
                    const T ezp = c ? (a ? EZp[b].y : EZp[b].x) : (a ? E[b][1].y : E[b][1].x);
                    T sm = 0;
                    sm = sm + (i > 0 ? txm * exm : T(0));
                    sm = sm + (i < n0 - 1 ? txp * exp : T(0));
                    sm = sm + (j > 0 ? tym * eym : T(0));
                    sm = sm + (j < n1 - 1 ? typ * eyp : T(0));
                    sm = sm + (k > 0 ? tzm * ezm : T(0));
                    sm = sm + (k < n2 - 1 ? tzp * ezp : T(0));
                    T d = txm + txp;
                    d = d + tym;
                    d = d + typ;
                    d = d + tzm;
                    d = d + tzp;
                    const T vol = (L.w[0][i] * L.w[1][j]) * L.w[2][k];
                    const T rv = a ? RR[b][c].y : RR[b][c].x;
                    const T rc = (rv - vol * mu) - (sm - d * ev);
                    const bool act = ((A[b][c] >> (8 * a)) & 0xff) != 0;
                    if (act) R += rc;
                }
        C.R[cid] = R;
        if (C.e) C.e[cid] = T(0);
        Rsum = (double)R;
    }
    double s = block_sum<256>(Rsum, sh, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// mu = sum(partials) / vol  (fixed order)
__global__ void k_finalize_mu(const double *partials, int n, const double *vol, double *mu) {
    __shared__ double sh[4];
    double s = 0.0;
    for (int q = threadIdx.x; q < n; q += 256) s += partials[q];
    s = block_sum<256>(s, sh, threadIdx.x);
    if (threadIdx.x == 0) *mu = (*vol > 0.0) ? s / *vol : 0.0;
}

// =======================================================================================
// coarse levels: red-black GS on  sum_F T_F (e_NB - e_C) = R_C - V_C mu
// =======================================================================================

// nsweeps red-black sweeps of a level of at most SMALL_LEVEL cells in one workgroup of 1024
// threads: each thread keeps the coefficients of up to SMALL_CPT cells in registers and the
// iterate lives in LDS, so a colour costs one LDS pass and one barrier instead of a launch.
// The arithmetic of every cell is that of launch_sweepC.
template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_smallC(Coarse<T> L, int nsweeps) {
    __shared__ T es[NT * SMALL_CPT];
    const int NC = L.n[0] * L.n[1] * L.n[2];
    const int sy = L.n[0], sz = L.n[0] * L.n[1];
    const T mu = (T)(*L.mu);
    // per cell: bit 0 live, 1 active, 2 colour, 3..8 neighbour present at -x,+x,-y,+y,-z,+z
    unsigned fl[SMALL_CPT];
    T txm[SMALL_CPT], txp[SMALL_CPT], tym[SMALL_CPT], typ[SMALL_CPT], tzm[SMALL_CPT], tzp[SMALL_CPT];
    T rhs[SMALL_CPT], dg[SMALL_CPT];
#pragma unroll
    for (int c = 0; c < SMALL_CPT; ++c) {
        const int id = (int)threadIdx.x + NT * c;
        const bool live = id < NC;
        const int idc = live ? id : 0;
        const int I = idc % L.n[0], J = (idc / L.n[0]) % L.n[1], K = idc / sz;
        const bool hx0 = I > 0, hx1 = I < L.n[0] - 1, hy0 = J > 0, hy1 = J < L.n[1] - 1, hz0 = K > 0,
                   hz1 = K < L.n[2] - 1;
        fl[c] = (live ? 1u : 0u) | ((live && L.active[idc] != 0) ? 2u : 0u) | ((unsigned)((I + J + K) & 1) << 2) |
                (hx0 ? 8u : 0u) | (hx1 ? 16u : 0u) | (hy0 ? 32u : 0u) | (hy1 ? 64u : 0u) | (hz0 ? 128u : 0u) |
                (hz1 ? 256u : 0u);
        txm[c] = L.Tl[0][idc];
        txp[c] = hx1 ? L.Tl[0][idc + 1] : T(0);
        tym[c] = L.Tl[1][idc];
        typ[c] = hy1 ? L.Tl[1][idc + sy] : T(0);
        tzm[c] = L.Tl[2][idc];
        tzp[c] = hz1 ? L.Tl[2][idc + sz] : T(0);
        const T v = (L.w[0][I] * L.w[1][J]) * L.w[2][K];
        rhs[c] = L.R[idc] - v * mu;
        T d = txm[c] + txp[c];
        d = d + tym[c];
        d = d + typ[c];
        d = d + tzm[c];
        d = d + tzp[c];
        dg[c] = d;
        if (live) es[id] = L.e[id];
    }
    __syncthreads();
    for (int sw = 0; sw < nsweeps; ++sw) {
        for (unsigned col = 0; col < 2; ++col) {
#pragma unroll
            for (int c = 0; c < SMALL_CPT; ++c) {
                const int id = (int)threadIdx.x + NT * c;
                const unsigned f = fl[c];
                if ((f & 2u) && ((f >> 2) & 1u) == col && dg[c] > T(0)) {
                    T num = 0;
                    num = num + ((f & 8u) ? txm[c] * es[id - 1] : T(0));
                    num = num + ((f & 16u) ? txp[c] * es[id + 1] : T(0));
                    num = num + ((f & 32u) ? tym[c] * es[id - sy] : T(0));
                    num = num + ((f & 64u) ? typ[c] * es[id + sy] : T(0));
                    num = num + ((f & 128u) ? tzm[c] * es[id - sz] : T(0));
                    num = num + ((f & 256u) ? tzp[c] * es[id + sz] : T(0));
                    es[id] = (num - rhs[c]) / dg[c];
                }
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int c = 0; c < SMALL_CPT; ++c) {
        const int id = (int)threadIdx.x + NT * c;
        if (fl[c] & 1u) L.e[id] = es[id];
    }
}

// the smallest workgroup that holds the level (one wave for the tiny levels, where barriers
// are nearly free)
template <typename T>
static void launch_smallC(const Coarse<T> &L, int64_t ncell, int nsweeps, hipStream_t s) {
    if (ncell <= 64 * SMALL_CPT)
        hipLaunchKernelGGL((k_smallC<T, 64>), dim3(1), dim3(64), 0, s, L, nsweeps);
    else if (ncell <= 256 * SMALL_CPT)
        hipLaunchKernelGGL((k_smallC<T, 256>), dim3(1), dim3(256), 0, s, L, nsweeps);
    else
        hipLaunchKernelGGL((k_smallC<T, 1024>), dim3(1), dim3(1024), 0, s, L, nsweeps);
}

template <typename T>
__global__ void __launch_bounds__(1024) k_coarsest(Coarse<T> L, int nsweeps, const double *vol) {
    __shared__ double sh[16];
    const int64_t NC = (int64_t)L.n[0] * L.n[1] * L.n[2];
    const T mu = (T)(*L.mu);
    for (int s = 0; s < nsweeps; ++s) {
        for (int colour = 0; colour < 2; ++colour) {
            for (int64_t id = threadIdx.x; id < NC; id += 1024) {
                int I, J, K;
                unflatten(id, L.n[0], L.n[1], I, J, K);
                if (((I + J + K) & 1) != colour || !L.active[id]) continue;
                T num, diag;
                coarse_stencil(L, L.e, I, J, K, id, num, diag);
                if (diag > T(0)) {
                    const T v = (L.w[0][I] * L.w[1][J]) * L.w[2][K];
                    L.e[id] = (num - (L.R[id] - v * mu)) / diag;
                }
            }
            __syncthreads();
        }
    }
    double acc = 0.0;
    for (int64_t id = threadIdx.x; id < NC; id += 1024) {
        if (!L.active[id]) continue;
        int I, J, K;
        unflatten(id, L.n[0], L.n[1], I, J, K);
        acc += (double)((L.w[0][I] * L.w[1][J]) * L.w[2][K]) * (double)L.e[id];
    }
    __shared__ double mean;
    double tot = block_sum<1024>(acc, sh, threadIdx.x);
    if (threadIdx.x == 0) mean = (*vol > 0.0) ? tot / *vol : 0.0;
    __syncthreads();
    const T m = (T)mean;
    for (int64_t id = threadIdx.x; id < NC; id += 1024)
        if (L.active[id]) L.e[id] -= m;
}

// prolongation with correction on a coarse level l from l+1: e_l += P e_{l+1} on active
// cells (trilinear in physical coordinates, or the parent's value when a contributing
// coarse cell is inactive)
template <typename T>
__device__ __forceinline__ double prolong_value(const Coarse<T> &C, const ProlongTab &P, int i, int j, int k) {
    const int ix[2] = {P.lo[0][i], P.hi[0][i]}, iy[2] = {P.lo[1][j], P.hi[1][j]}, iz[2] = {P.lo[2][k], P.hi[2][k]};
    const double tx = P.t[0][i], ty = P.t[1][j], tz = P.t[2][k];
    const double wx[2] = {1.0 - tx, tx}, wy[2] = {1.0 - ty, ty}, wz[2] = {1.0 - tz, tz};
    const bool two[3] = {ix[0] != ix[1], iy[0] != iy[1], iz[0] != iz[1]};
    bool all = true;
    double s = 0.0;
    // fixed 2x2x2 loop (a second contributor that coincides with the first is skipped),
    // unrolled so that all coarse loads are issued together
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const bool ok = (a == 0 || two[0]) && (b == 0 || two[1]) && (c == 0 || two[2]);
                const int64_t cid = ((int64_t)iz[c] * C.n[1] + iy[b]) * C.n[0] + ix[a];
                const bool act = C.active[cid] != 0;
                const double term = (wx[a] * wy[b]) * wz[c] * (double)C.e[cid];
                if (ok) {
                    if (!act) all = false;
                    s += term;
                }
            }
    if (!all) {  // the parent: the first contributor on every axis
        const int pi = P.lo[0][i], pj = P.lo[1][j], pk = P.lo[2][k];
        s = (double)C.e[((int64_t)pk * C.n[1] + pj) * C.n[0] + pi];
    }
    return s;
}

template <typename T>
__global__ void k_prolongC(Coarse<T> L, Coarse<T> C, ProlongTab P) {
    const int64_t N = (int64_t)L.n[0] * L.n[1] * L.n[2];
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N || !L.active[id]) return;
    int i, j, k;
    unflatten(id, L.n[0], L.n[1], i, j, k);
    L.e[id] = (T)((double)L.e[id] + prolong_value(C, P, i, j, k));
}

// The same for any child map, on large levels, with the coarser values staged in LDS: the
// tiling and the ring of coarser planes of the level-0 prolongation k_prolong0_lds (a
// workgroup's 64 x 4 columns draw on at most PLC_CW x PLC_CH coarser columns; each coarser
// plane it needs is read once, values and activity, the next one while the current plane is
// computed).  Per cell the terms, their order and the fallback to the parent are those of
// prolong_value, so the result is bitwise that of k_prolongC.
constexpr int PLC_CW = 68, PLC_CH = 6, PLC_RING = 4, PLC_PER = (PLC_CW * PLC_CH + ZM_NT - 1) / ZM_NT;
constexpr int64_t PROLONG_LDS_MIN_CELLS = 1 << 18;

template <typename T>
__global__ void __launch_bounds__(ZM_NT) k_prolongC_lds(Coarse<T> L, Coarse<T> C, ProlongTab P, ZTiles t) {
    __shared__ T ec[PLC_RING][PLC_CH][PLC_CW];
    __shared__ uint8_t ca[PLC_RING][PLC_CH][PLC_CW];
    const ZPos z = zpos(t, L.n[2]);
    if (!z.live) return;
    const int nx = L.n[0], ny = L.n[1], nz = L.n[2];
    const bool in = z.i < nx && z.j < ny;
    const int ic = min(z.i, nx - 1), jc = min(z.j, ny - 1);
    const int64_t plane = (int64_t)nx * ny, rowoff = (int64_t)jc * nx + ic;
    // the tile's coarser window (tables are monotone: lo non-decreasing, hi = lo or lo +- 1)
    const int ia = min(z.i - z.lane, nx - 1), ib = min(z.i - z.lane + ZM_TX - 1, nx - 1);
    const int ja = min(z.j - z.wave, ny - 1), jb = min(z.j - z.wave + ZM_TY - 1, ny - 1);
    const int cx0 = min(P.lo[0][ia], P.hi[0][ia]), cx1 = max(P.lo[0][ib], P.hi[0][ib]);
    const int cy0 = min(P.lo[1][ja], P.hi[1][ja]), cy1 = max(P.lo[1][jb], P.hi[1][jb]);
    const int cw = cx1 - cx0 + 1, ch = cy1 - cy0 + 1;
    const int ix[2] = {P.lo[0][ic] - cx0, P.hi[0][ic] - cx0}, iy[2] = {P.lo[1][jc] - cy0, P.hi[1][jc] - cy0};
    const double tx = P.t[0][ic], ty = P.t[1][jc];
    const double wx[2] = {1.0 - tx, tx}, wy[2] = {1.0 - ty, ty};
    const bool twox = ix[0] != ix[1], twoy = iy[0] != iy[1];
    const int64_t cny = C.n[1], cnx = C.n[0];
    // coarser values and activity this thread stages for one coarser plane
    auto cload = [=](int K, T (&v)[PLC_PER], uint8_t (&a)[PLC_PER]) {
#pragma unroll
        for (int q = 0; q < PLC_PER; ++q) {
            const int e = (int)threadIdx.x + q * ZM_NT;
            const int r = e / PLC_CW, c = e % PLC_CW;
            const bool ok = r < ch && c < cw;
            const int64_t id = ((int64_t)K * cny + cy0 + min(r, ch - 1)) * cnx + cx0 + min(c, cw - 1);
            v[q] = ok ? C.e[id] : T(0);
            a[q] = ok ? C.active[id] : (uint8_t)0;
        }
    };
    auto cstore = [&](int K, const T (&v)[PLC_PER], const uint8_t (&a)[PLC_PER]) {
#pragma unroll
        for (int q = 0; q < PLC_PER; ++q) {
            const int e = (int)threadIdx.x + q * ZM_NT;
            if (e < PLC_CW * PLC_CH) {
                ec[K & (PLC_RING - 1)][e / PLC_CW][e % PLC_CW] = v[q];
                ca[K & (PLC_RING - 1)][e / PLC_CW][e % PLC_CW] = a[q];
            }
        }
    };
    auto need_hi = [=](int k) { return max(P.lo[2][k], P.hi[2][k]); };
    const int k0 = z.k0, k1 = z.k1;
    int have;  // highest coarser plane staged
    {
        const int a = min(P.lo[2][k0], P.hi[2][k0]), b = need_hi(k0);
        T v[PLC_PER];
        uint8_t av[PLC_PER];
        for (int K = a; K <= b; ++K) {
            cload(K, v, av);
            cstore(K, v, av);
        }
        have = b;
        __syncthreads();
    }
    T ecur = L.e[(int64_t)k0 * plane + rowoff];
    uint8_t acur = L.active[(int64_t)k0 * plane + rowoff];
    for (int k = k0; k < k1; ++k) {
        const int64_t nbase = (int64_t)min(k + 1, nz - 1) * plane + rowoff;
        const T enext = L.e[nbase];
        const uint8_t anext = L.active[nbase];
        // the next plane needs at most one more coarser plane: load it now, stage it after
        const int nb = (k + 1 < nz) ? need_hi(k + 1) : have;
        const bool more = nb > have;
        T v[PLC_PER];
        uint8_t av[PLC_PER];
        if (more) cload(nb, v, av);
        const int iz[2] = {P.lo[2][k], P.hi[2][k]};
        const double tz = P.t[2][k];
        const double wz[2] = {1.0 - tz, tz};
        const bool twoz = iz[0] != iz[1];
        bool all = true;
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const bool ok = (a == 0 || twox) && (b == 0 || twoy) && (c == 0 || twoz);
                    const int r = iz[c] & (PLC_RING - 1);
                    const double term = (wx[a] * wy[b]) * wz[c] * (double)ec[r][iy[b]][ix[a]];
                    if (ok) {
                        if (!ca[r][iy[b]][ix[a]]) all = false;
                        s += term;
                    }
                }
        if (!all) s = (double)ec[iz[0] & (PLC_RING - 1)][iy[0]][ix[0]];
        if (in && acur) L.e[(int64_t)k * plane + rowoff] = (T)((double)ecur + s);
        if (more) {
            __syncthreads();  // every thread is done with the slot the new plane goes to
            cstore(nb, v, av);
            have = nb;
        }
        __syncthreads();
        ecur = enext;
        acur = anext;
    }
}

// The same for a level pair with every axis halved: a thread per coarse cell updates its
// 2 x 2 x 2 children, loaded and stored as x pairs.  On a halved axis the first contributor
// of a child is its parent and the second (if any) the parent's neighbour on the child's
// side (the table's hi), so the 3 x 3 x 3 coarse neighbourhood, loaded once, holds every
// contributor.  Per child the terms, their order and the fallback to the parent are those
// of prolong_value, so the result is bitwise that of k_prolongC.
// Smaller levels keep k_prolongC: there the longer load chain of a thread outweighs the
// coalescing (64^3 from 32^3: 6.8 us against 6.4; 128^3 from 64^3: 13 us against 22).
constexpr int64_t PROLONG8_MIN_CELLS = 1 << 19;
template <typename T>
__global__ void __launch_bounds__(256) k_prolongC8(Coarse<T> L, Coarse<T> C, ProlongTab P) {
    using V = typename Pair2<T>::type;
    const int64_t NC = (int64_t)C.n[0] * C.n[1] * C.n[2];
    const int64_t cid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (cid >= NC) return;
    int I, J, K;
    unflatten(cid, C.n[0], C.n[1], I, J, K);
    const int m0 = C.n[0], m1 = C.n[1], m2 = C.n[2];
    const int64_t csy = m0, csz = (int64_t)m0 * m1;
    // coarse neighbourhood, indices clamped (a clamped entry is never a contributor)
    double ce[3][3][3];
    uint32_t ca = 0;  // bit (dz*9 + dy*3 + dx): active
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const int x = min(max(I + dx - 1, 0), m0 - 1), y = min(max(J + dy - 1, 0), m1 - 1),
                          z = min(max(K + dz - 1, 0), m2 - 1);
                const int64_t q = (int64_t)z * csz + (int64_t)y * csy + x;
                ce[dz][dy][dx] = (double)C.e[q];
                ca |= (C.active[q] != 0 ? 1u : 0u) << (dz * 9 + dy * 3 + dx);
            }
    // per child side (0: low, 1: high) and axis: has a second contributor, and its weight
    const int i0 = 2 * I, j0 = 2 * J, k0 = 2 * K;
    bool two[3][2];
    double tw[3][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        two[0][h] = P.lo[0][i0 + h] != P.hi[0][i0 + h];
        two[1][h] = P.lo[1][j0 + h] != P.hi[1][j0 + h];
        two[2][h] = P.lo[2][k0 + h] != P.hi[2][k0 + h];
        tw[0][h] = P.t[0][i0 + h];
        tw[1][h] = P.t[1][j0 + h];
        tw[2][h] = P.t[2][k0 + h];
    }
    const int n0 = L.n[0];
    const int64_t sy = n0, sz = (int64_t)n0 * L.n[1];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t row = (int64_t)(k0 + c) * sz + (int64_t)(j0 + b) * sy + i0;
            V ev = *reinterpret_cast<const V *>(L.e + row);
            const uint16_t fa = *reinterpret_cast<const uint16_t *>(L.active + row);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const double wx[2] = {1.0 - tw[0][a], tw[0][a]}, wy[2] = {1.0 - tw[1][b], tw[1][b]},
                             wz[2] = {1.0 - tw[2][c], tw[2][c]};
                // neighbourhood index of contributor (lo, hi) on each axis: 1 is the parent
                const int hx = a ? 2 : 0, hy = b ? 2 : 0, hz = c ? 2 : 0;
                bool all = true;
                double sv = 0.0;
#pragma unroll
                for (int cz = 0; cz < 2; ++cz)
#pragma unroll
                    for (int cy = 0; cy < 2; ++cy)
#pragma unroll
                        for (int cx = 0; cx < 2; ++cx) {
                            const bool ok = (cx == 0 || two[0][a]) && (cy == 0 || two[1][b]) && (cz == 0 || two[2][c]);
                            const int ox = cx ? hx : 1, oy = cy ? hy : 1, oz = cz ? hz : 1;
                            const bool act = (ca >> (oz * 9 + oy * 3 + ox)) & 1u;
                            const double term = (wx[cx] * wy[cy]) * wz[cz] * ce[oz][oy][ox];
                            if (ok) {
                                if (!act) all = false;
                                sv += term;
                            }
                        }
                if (!all) sv = ce[1][1][1];
                const bool fine_act = ((fa >> (8 * a)) & 0xff) != 0;
                T &dst = a ? ev.y : ev.x;
                if (fine_act) dst = (T)((double)dst + sv);
            }
            *reinterpret_cast<V *>(L.e + row) = ev;
        }
}

// =======================================================================================
// residual norm on level 0 with the lambda update
//   r = f - S p (fluid rows);  a = r - lambda_k;  partials of sum V a, sum a^2, sum a
//   lambda_{k+1} = lambda_k + delta, delta = sum V a / sum V
//   ||r - lambda_{k+1}||^2 = sum a^2 - 2 delta sum a + delta^2 n_fluid
// WRITE_R32: also store the FP32 right-hand side a for the mixed-precision inner cycle
// =======================================================================================

constexpr int NORM_NT = 256;

template <bool WRITE_R32>
__global__ void __launch_bounds__(NORM_NT) k_norm0(Fine<double> F, const double *__restrict__ p,
                                                   const double *__restrict__ f, const double *__restrict__ lamp,
                                                   float *r32, double *partials) {
    const int64_t N = (int64_t)F.nx * F.ny * F.nz;
    const double lam = *lamp;
    double sv = 0.0, s2 = 0.0, s1 = 0.0;
    for (int64_t id = (int64_t)blockIdx.x * NORM_NT + threadIdx.x; id < N; id += (int64_t)gridDim.x * NORM_NT) {
        if (F.type[id] != T_FLUID) {
            if (WRITE_R32) r32[id] = 0.0f;
            continue;
        }
        int i, j, k;
        unflatten(id, F.nx, F.ny, i, j, k);
        double num, diag;
        fine_stencil(F, p, i, j, k, id, num, diag);
        const double r = f[id] - (num - diag * p[id]);
        const double a = r - lam;
        sv += ((F.wx[i] * F.wy[j]) * F.wz[k]) * a;
        s2 += a * a;
        s1 += a;
        if (WRITE_R32) r32[id] = (float)a;
    }
    double sums[3] = {sv, s2, s1};
    block_sums_store<NORM_NT, 3>(sums, partials);
}

// The kernels that add up partials: one workgroup of FIN_NT threads, bound by the round trips of
// its loads, so every thread has only a few (256 threads and one sum at a time: 5.4 us).
constexpr int FIN_NT = 1024;

// sums of the NS-tuples a[0 .. nb); v[q] is the sum in thread 0
template <int NS>
__device__ __forceinline__ void sum_partials(const double *a, int nb, double (&v)[NS]) {
    for (int q = threadIdx.x; q < nb; q += FIN_NT) {
#pragma unroll
        for (int c = 0; c < NS; ++c) v[c] += a[NS * q + c];
    }
}
template <int NS>
__device__ __forceinline__ void finish_sums(double (&v)[NS]) {
    __shared__ double sh[FIN_NT / 64][NS], tot[NS];
    block_sums<FIN_NT, NS>(v, sh, threadIdx.x);
#pragma unroll
    for (int c = 0; c < NS; ++c)
        if ((int)threadIdx.x == c) tot[c] = v[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NS; ++c) v[c] = tot[c];
}

__global__ void __launch_bounds__(FIN_NT) k_norm_finalize(const double *partials, int nb, Scalars *sc, double nfluid,
                                                          int set_ref) {
    double v[3] = {0.0, 0.0, 0.0};
    sum_partials<3>(partials, nb, v);
    finish_sums<3>(v);
    if (threadIdx.x == 0) {
        const double a = v[0], b = v[1], c = v[2];
        const double delta = a / sc->vol[0];
        double q2 = b - 2.0 * delta * c + delta * delta * nfluid;
        if (q2 < 0.0) q2 = 0.0;
        const double nrm = sqrt(q2);
        sc->lambda = sc->lambda + delta;
        sc->delta = delta;
        sc->delta32 = (float)delta;
        sc->norm = nrm;
        if (set_ref) sc->ref = nrm;
        sc->rel = (sc->ref > 0.0) ? nrm / sc->ref : 0.0;
        if (!isfinite(nrm) || !isfinite(sc->lambda)) sc->bad = 1;
    }
}

// reference norm ||f - Vmean(f)|| over fluid cells (two passes: mean, then deviations)
__global__ void __launch_bounds__(NORM_NT) k_fsum(Fine<double> F, const double *__restrict__ f, const double *meanp,
                                                  double *partials, int pass) {
    __shared__ double sh[NORM_NT / 64];
    const int64_t N = (int64_t)F.nx * F.ny * F.nz;
    const double mean = pass ? *meanp : 0.0;
    double s = 0.0;
    for (int64_t id = (int64_t)blockIdx.x * NORM_NT + threadIdx.x; id < N; id += (int64_t)gridDim.x * NORM_NT) {
        if (F.type[id] != T_FLUID) continue;
        if (pass == 0) {
            int i, j, k;
            unflatten(id, F.nx, F.ny, i, j, k);
            s += ((F.wx[i] * F.wy[j]) * F.wz[k]) * f[id];
        } else {
            const double d = f[id] - mean;
            s += d * d;
        }
    }
    double t = block_sum<NORM_NT>(s, sh, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ void __launch_bounds__(FIN_NT) k_fsum_finalize(const double *partials, int nb, Scalars *sc, int pass) {
    double v[1] = {0.0};
    sum_partials<1>(partials, nb, v);
    finish_sums<1>(v);
    if (threadIdx.x == 0) {
        if (pass == 0) sc->vmean = v[0] / sc->vol[0];
        else sc->ref = sqrt(v[0]);
    }
}

// volume-weighted mean of p over fluid cells, then pdst = pcur - mean (fluid, ghost), 0 (dead)
__global__ void __launch_bounds__(NORM_NT) k_psum(Fine<double> F, const double *__restrict__ p, double *partials) {
    __shared__ double sh[NORM_NT / 64];
    const int64_t N = (int64_t)F.nx * F.ny * F.nz;
    double s = 0.0;
    for (int64_t id = (int64_t)blockIdx.x * NORM_NT + threadIdx.x; id < N; id += (int64_t)gridDim.x * NORM_NT) {
        if (F.type[id] != T_FLUID) continue;
        int i, j, k;
        unflatten(id, F.nx, F.ny, i, j, k);
        s += ((F.wx[i] * F.wy[j]) * F.wz[k]) * p[id];
    }
    double t = block_sum<NORM_NT>(s, sh, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ void k_shift(const uint8_t *__restrict__ type, int64_t N, const double *__restrict__ pcur, double *pdst,
                        const Scalars *sc) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    const double m = sc->vmean;
    pdst[id] = (type[id] == T_DEAD) ? 0.0 : pcur[id] - m;
}

// =======================================================================================
// launchers
// =======================================================================================

hipError_t sweep0_f64(ibm_grid *g, const double *pin, double *pout, const double *f, const double *lambda,
                      hipStream_t s) {
    return launch_sweep<double>(fine64(g), pin, pout, f, lambda, s);
}

hipError_t refresh_f64(ibm_grid *g, const double *src_ghost, double *dst, hipStream_t s) {
    return launch_refresh<double>(g, src_ghost, dst, g->g_h, s);
}

template <typename T>
__global__ void k_apply0(Fine<T> F, const T *__restrict__ p, T *out) {
    const int64_t N = (int64_t)F.nx * F.ny * F.nz;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    if (F.type[id] != T_FLUID) {
        out[id] = T(0);
        return;
    }
    int i, j, k;
    unflatten(id, F.nx, F.ny, i, j, k);
    T num, diag;
    fine_stencil(F, p, i, j, k, id, num, diag);
    out[id] = num - diag * p[id];
}

hipError_t apply0_f64(ibm_grid *g, const double *p, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_apply0<double>, dim3((unsigned)((g->N + 255) / 256)), dim3(256), 0, s, fine64(g), p, out);
    return hipGetLastError();
}

static int nblk(int64_t n, int nt = 256) { return (int)((n + nt - 1) / nt); }

template <typename T>
struct FineOf;
template <>
struct FineOf<double> {
    static Fine<double> get(ibm_grid *g) { return fine64(g); }
};
template <>
struct FineOf<float> {
    static Fine<float> get(ibm_grid *g) { return fine32(g); }
};

// one V(nu1, nu2) cycle in precision T on level 0.
// bufs[0..1]: the two level-0 buffers, *cur: index of the current iterate.
// rhs: level-0 right-hand side; lam: device scalar shift of the right-hand side;
// gh: right-hand sides of the ghost equations (nullptr: homogeneous error equation).
// level-0 sweep, timed by start and end events when profiling is on
template <typename T>
static hipError_t timed_sweep(ibm_grid *g, const Fine<T> &F, const T *pin, T *pout, const T *rhs, const T *lam,
                              hipStream_t s) {
    Prof &P = g->prof;
    const bool rec = P.on && (P.seq++ % P.stride) == 0 && P.used + 2 <= (int)P.ev.size();
    hipError_t e;
    // the runtime records the two events at the kernel's own start and end
    if ((e = launch_sweep<T>(F, pin, pout, rhs, lam, s, rec ? P.ev[P.used] : nullptr,
                             rec ? P.ev[P.used + 1] : nullptr)) != hipSuccess)
        return e;
    if (rec) {
        P.kind[P.used / 2] = (sizeof(T) == 8) ? 0 : 1;
        P.used += 2;
    }
    return hipSuccess;
}

// nsweeps red-black sweeps of coarse level l (more than SMALL_LEVEL cells), out of place between
// its two error buffers, which are swapped after each (every later view of the level sees the
// current one).  The first sweep forms mu when ms has its partials; zero: the correction is 0.
// (Levels swept by colours work in place, on a cleared correction, with mu formed by a launch.)
template <typename T>
static hipError_t smooth_level(ibm_grid *g, int l, int nsweeps, const MuSource &ms, bool zero, hipStream_t s) {
    LevelHost &H = g->lev[l];
    if (sweepC_by_colours(H.n)) {
        for (int q = 0; q < nsweeps; ++q) {
            const hipError_t e = launch_sweepC_colours<T>(coarse_view<T>(g, l), s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    for (int q = 0; q < nsweeps; ++q) {
        const hipError_t e = launch_sweepC<T>(coarse_view<T>(g, l), level_e2<T>(H), q == 0 ? ms : MuSource{},
                                              zero && q == 0, s);
        if (e != hipSuccess) return e;
        std::swap(level_e<T>(H), level_e2<T>(H));
    }
    return hipSuccess;
}

template <typename T>
static hipError_t vcycle_impl(ibm_grid *g, T **bufs, int *cur, const T *rhs, const T *lam, const double *gh,
                              const ibm_solve_opts *o, hipStream_t s, const T *start = nullptr,
                              double *wide = nullptr, bool swept = false) {
    // swept: the first pre-smoothing sweep and its ghost refresh are done, bufs[*cur] holds its result
    // start (requires nu1 > 0): the iterate the first pre-smoothing sweep reads instead of
    // bufs[*cur]; it is only read, and the sweeps continue in bufs
    // wide (FP32 cycle with nu2 > 0): the last post-smoothing sweep and its ghost refresh
    // write the result widened to FP64 there instead of into bufs (that sweep is not timed:
    // it moves 17 bytes per cell, not 13)
    const Fine<T> F = FineOf<T>::get(g);
    hipError_t e;
    for (int q = swept ? 1 : 0; q < o->nu1; ++q) {
        T *pin = (q == 0 && start) ? const_cast<T *>(start) : bufs[*cur], *pout = bufs[1 - *cur];
        if ((e = timed_sweep<T>(g, F, pin, pout, rhs, lam, s)) != hipSuccess) return e;
        if ((e = launch_refresh<T>(g, pin, pout, gh, s)) != hipSuccess) return e;
        *cur = 1 - *cur;
    }
    if (g->nlev > 1) {
        const int Lc = g->nlev - 1;
        const int lt = tail_first(g->lev, g->nlev);
        const bool tail = lt <= Lc;
        const int Lb = tail ? lt : Lc;  // levels 1 .. Lb-1 run level by level
        int nparts = 0;                 // restriction partials into level Lb
        // levels whose first sweep takes a zero correction without reading it (not cleared then)
        auto level_swept = [&](int l) {
            return l < Lb && g->lev[l].ncell() > SMALL_LEVEL && o->nu1 > 0 && !sweepC_by_colours(g->lev[l].n);
        };
        {
            Coarse<T> C1 = coarse_view<T>(g, 1);
            if (level_swept(1)) C1.e = nullptr;
            if ((e = launch_restrict0<T>(F, bufs[*cur], rhs, lam, C1, child_map(g->lev[1]), g->partials, &nparts,
                                         s)) != hipSuccess)
                return e;
        }
        // mu of level l from the partials of the restriction into it: by its first sweep where one
        // follows and the partials are few for it, by the tail for its own levels, else by a launch
        auto mu_by_sweep = [&](int l) { return level_swept(l) && sweepC_forms_mu<T>(g->lev[l].n, nparts); };
        auto finalize_mu = [&](int l) {
            if (!mu_by_sweep(l) && !(tail && l == lt))
                hipLaunchKernelGGL(k_finalize_mu, dim3(1), dim3(256), 0, s, g->partials, nparts, &g->sc->vol[l],
                                   &g->sc->mu[l]);
        };
        finalize_mu(1);
        for (int l = 1; l < Lb; ++l) {
            if (g->lev[l].ncell() <= SMALL_LEVEL) {
                if (o->nu1 > 0) launch_smallC<T>(coarse_view<T>(g, l), g->lev[l].ncell(), o->nu1, s);
            } else {
                MuSource ms;
                ms.partials = g->partials;
                ms.n = mu_by_sweep(l) ? nparts : 0;
                ms.vol = &g->sc->vol[l];
                ms.mu = &g->sc->mu[l];
                if ((e = smooth_level<T>(g, l, o->nu1, ms, true, s)) != hipSuccess) return e;
            }
            Coarse<T> L = coarse_view<T>(g, l);  // after the sweeps: the current error buffer
            Coarse<T> C = coarse_view<T>(g, l + 1);
            if (level_swept(l + 1)) C.e = nullptr;
            const ChildMap M = child_map(g->lev[l + 1]);
            int nbc = nblk(g->lev[l + 1].ncell());
            if (M.halved[0] && M.halved[1] && M.halved[2]) {
                hipLaunchKernelGGL(k_resrestrictC8<T>, dim3(nbc), dim3(256), 0, s, L, C, g->partials);
            } else {
                RowTiles t;
                if ((e = row_tiles(M, C.n, zmarch_partials_max(g->nx, g->ny, g->nz), &t, &nbc)) != hipSuccess)
                    return e;
                auto k = L.n[2] == 1 ? k_resrestrictC_map<T, true> : k_resrestrictC_map<T, false>;
                hipLaunchKernelGGL(k, dim3(nbc), dim3(RM_NT), 0, s, L, C, M, t, g->partials);
            }
            nparts = nbc;
            finalize_mu(l + 1);
        }
        if (tail) {
            if ((e = launch_tail<T>(g, lt, coarse_view<T>(g, lt), nparts, o, s)) != hipSuccess) return e;
        } else {  // a coarsest level of more than SMALL_LEVEL cells
            hipLaunchKernelGGL(k_coarsest<T>, dim3(1), dim3(1024), 0, s, coarse_view<T>(g, Lc), o->coarsest_sweeps,
                               &g->sc->vol[Lc]);
        }
        for (int l = Lb - 1; l >= 1; --l) {
            Coarse<T> L = coarse_view<T>(g, l);
            int nb = nblk(g->lev[l].ncell());
            const ProlongTab PT = prolong_tab(g, l);
            if (PT.halved[0] && PT.halved[1] && PT.halved[2] && g->lev[l].prolong_sides &&
                g->lev[l].ncell() >= PROLONG8_MIN_CELLS)
                hipLaunchKernelGGL(k_prolongC8<T>, dim3(nblk(g->lev[l + 1].ncell())), dim3(256), 0, s, L,
                                   coarse_view<T>(g, l + 1), PT);
            else if (g->lev[l].ncell() >= PROLONG_LDS_MIN_CELLS) {
                const ZTiles t = ztiles(L.n[0], L.n[1], L.n[2]);
                hipLaunchKernelGGL(k_prolongC_lds<T>, dim3(t.grid), dim3(ZM_NT), 0, s, L, coarse_view<T>(g, l + 1), PT,
                                   t);
            } else
                hipLaunchKernelGGL(k_prolongC<T>, dim3(nb), dim3(256), 0, s, L, coarse_view<T>(g, l + 1), PT);
            if (g->lev[l].ncell() <= SMALL_LEVEL) {
                if (o->nu2 > 0) launch_smallC<T>(L, g->lev[l].ncell(), o->nu2, s);
            } else if ((e = smooth_level<T>(g, l, o->nu2, MuSource{}, false, s)) != hipSuccess) {
                return e;
            }
        }
        {
            T *pin = bufs[*cur], *pout = bufs[1 - *cur];
            if ((e = launch_prolong0<T>(F, pin, pout, coarse_view<T>(g, 1), prolong_tab(g, 0), s)) != hipSuccess)
                return e;
            if ((e = launch_refresh<T>(g, pin, pout, gh, s)) != hipSuccess) return e;
            *cur = 1 - *cur;
        }
    }
    for (int q = 0; q < o->nu2; ++q) {
        T *pin = bufs[*cur], *pout = bufs[1 - *cur];
        if constexpr (std::is_same<T, float>::value) {
            if (wide && q + 1 == o->nu2) {
                if ((e = launch_sweep_widen(F, pin, wide, rhs, lam, s)) != hipSuccess) return e;
                return launch_refresh_widen(g, pin, wide, gh, s);
            }
        }
        if ((e = timed_sweep<T>(g, F, pin, pout, rhs, lam, s)) != hipSuccess) return e;
        if ((e = launch_refresh<T>(g, pin, pout, gh, s)) != hipSuccess) return e;
        *cur = 1 - *cur;
    }
    return hipGetLastError();
}

hipError_t vcycle_f64(ibm_grid *g, double **bufs, int *cur, const double *f, hipStream_t s, const ibm_solve_opts *o,
                      bool swept) {
    return vcycle_impl<double>(g, bufs, cur, f, &g->sc->lambda, g->g_h, o, s, nullptr, nullptr, swept);
}

hipError_t vcycle_ahead(ibm_grid *g, double **bufs, int *cur, const double *f, hipStream_t s) {
    double *pin = bufs[*cur], *pout = bufs[1 - *cur];
    const hipError_t e = launch_sweep<double>(fine64(g), pin, pout, f, &g->sc->lambda, s);
    if (e != hipSuccess) return e;
    *cur = 1 - *cur;
    return launch_refresh<double>(g, pin, pout, g->g_h, s);
}

// e32 := 0 (dead cells too), so the inner cycle starts from a zero correction
__global__ void k_zero32(float *a, float *b, int64_t N) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    a[id] = 0.0f;
    b[id] = 0.0f;
}

// p_next = p_cur + e on fluid cells (FP64 update of the refinement step)
__global__ void k_add_correction(const uint8_t *__restrict__ type, int64_t N, const double *__restrict__ pcur,
                                 const float *__restrict__ e, double *pnext) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N || type[id] != T_FLUID) return;
    pnext[id] = pcur[id] + (double)e[id];
}

// one mixed-precision refinement step: the FP32 right-hand side r32 = r - lambda_k was
// written by the preceding FP64 norm pass and delta32 = lambda_{k+1} - lambda_k; solve
// S e = r32 - delta with one FP32 V-cycle from e = 0, then p += e and an FP64 ghost refresh
hipError_t vcycle_mixed(ibm_grid *g, double **bufs, int *cur, const double *f, hipStream_t s,
                        const ibm_solve_opts *o) {
    (void)f;
    hipError_t e;
    hipLaunchKernelGGL(k_zero32, dim3(nblk(g->N)), dim3(256), 0, s, g->e32a, g->e32b, g->N);
    float *eb[2] = {g->e32a, g->e32b};
    int ecur = 0;
    if ((e = vcycle_impl<float>(g, eb, &ecur, g->r32, &g->sc->delta32, nullptr, o, s)) != hipSuccess) return e;
    double *pin = bufs[*cur], *pout = bufs[1 - *cur];
    hipLaunchKernelGGL(k_add_correction, dim3(nblk(g->N)), dim3(256), 0, s, g->type, g->N, pin, eb[ecur], pout);
    if ((e = launch_refresh<double>(g, pin, pout, g->g_h, s)) != hipSuccess) return e;
    *cur = 1 - *cur;
    return hipGetLastError();
}

hipError_t norm_pass(ibm_grid *g, const double *p, const double *f, hipStream_t s, bool write_r32, bool first) {
    if (write_r32)
        hipLaunchKernelGGL(k_norm0<true>, dim3(red_blocks(g->N)), dim3(NORM_NT), 0, s, fine64(g), p, f, &g->sc->lambda, g->r32,
                           g->partials);
    else
        hipLaunchKernelGGL(k_norm0<false>, dim3(red_blocks(g->N)), dim3(NORM_NT), 0, s, fine64(g), p, f, &g->sc->lambda,
                           (float *)nullptr, g->partials);
    hipLaunchKernelGGL(k_norm_finalize, dim3(1), dim3(FIN_NT), 0, s, g->partials, red_blocks(g->N), g->sc, (double)g->nfluid,
                       0);
    (void)first;
    return hipGetLastError();
}

hipError_t ref_norm_pass(ibm_grid *g, const double *f, hipStream_t s) {
    hipLaunchKernelGGL(k_fsum, dim3(red_blocks(g->N)), dim3(NORM_NT), 0, s, fine64(g), f, &g->sc->vmean, g->partials, 0);
    hipLaunchKernelGGL(k_fsum_finalize, dim3(1), dim3(FIN_NT), 0, s, g->partials, red_blocks(g->N), g->sc, 0);
    hipLaunchKernelGGL(k_fsum, dim3(red_blocks(g->N)), dim3(NORM_NT), 0, s, fine64(g), f, &g->sc->vmean, g->partials, 1);
    hipLaunchKernelGGL(k_fsum_finalize, dim3(1), dim3(FIN_NT), 0, s, g->partials, red_blocks(g->N), g->sc, 1);
    return hipGetLastError();
}

hipError_t gauge_pass(ibm_grid *g, const double *pcur, double *pdst, hipStream_t s) {
    hipLaunchKernelGGL(k_psum, dim3(red_blocks(g->N)), dim3(NORM_NT), 0, s, fine64(g), pcur, g->partials);
    hipLaunchKernelGGL(k_fsum_finalize, dim3(1), dim3(FIN_NT), 0, s, g->partials, red_blocks(g->N), g->sc, 0);
    hipLaunchKernelGGL(k_shift, dim3(nblk(g->N)), dim3(256), 0, s, g->type, g->N, pcur, pdst, g->sc);
    return hipGetLastError();
}

// start of a solve: both buffers hold the initial iterate on fluid and ghost cells (zero
// unless a guess is given) and 0 on dead cells; then the ghosts of p2 are refreshed
__global__ void k_init(const uint8_t *__restrict__ type, int64_t N, double *p, double *p2, int use_guess) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    double v = (type[id] == T_DEAD || !use_guess) ? 0.0 : p[id];
    p[id] = v;
    p2[id] = v;
}

hipError_t init_solution(ibm_grid *g, double *p, double *p2, int use_guess, hipStream_t s) {
    hipLaunchKernelGGL(k_init, dim3(nblk(g->N)), dim3(256), 0, s, g->type, g->N, p, p2, use_guess);
    return launch_refresh<double>(g, p, p2, g->g_h, s);
}

// =======================================================================================
// projection: divergence right-hand side and velocity correction (MAC faces)
// =======================================================================================

__global__ void k_rhs(Fine<double> F, const double *__restrict__ u, const double *__restrict__ v,
                      const double *__restrict__ w, double dt, double *f) {
    const int64_t N = (int64_t)F.nx * F.ny * F.nz;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    if (F.type[id] != T_FLUID) {
        f[id] = 0.0;
        return;
    }
    const int nx = F.nx, ny = F.ny;
    int i, j, k;
    unflatten(id, nx, ny, i, j, k);
    const int64_t iu = ((int64_t)k * ny + j) * (nx + 1) + i;
    const int64_t iv = ((int64_t)k * (ny + 1) + j) * nx + i;
    const int64_t iw = ((int64_t)k * ny + j) * nx + i;
    double div = (u[iu + 1] - u[iu]) / F.wx[i];
    div = div + (v[iv + nx] - v[iv]) / F.wy[j];
    div = div + (w[iw + (int64_t)nx * ny] - w[iw]) / F.wz[k];
    f[id] = div / dt;
}

hipError_t rhs_pass(ibm_grid *g, const double *u, const double *v, const double *w, double dt, double *f,
                    hipStream_t s) {
    hipLaunchKernelGGL(k_rhs, dim3(nblk(g->N)), dim3(256), 0, s, fine64(g), u, v, w, dt, f);
    return hipGetLastError();
}

// u_f -= dt (p_nb - p_c)/d_f on interior faces with at least one fluid cell.  A thread owns
// cell (i, j, k) and corrects its three low faces (the cell reads p and its type once for
// all three); the low faces of the first cells and the high faces of the last cells along
// an axis are box walls and stay as they are.
__global__ void k_correct(const uint8_t *__restrict__ type, int nx, int ny, int nz, const double *__restrict__ dcx,
                          const double *__restrict__ dcy, const double *__restrict__ dcz, const double *__restrict__ p,
                          double dt, double *u, double *v, double *w) {
    const int64_t N = (int64_t)nx * ny * nz;
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= N) return;
    int i, j, k;
    unflatten(b, nx, ny, i, j, k);
    const bool fb = type[b] == T_FLUID;
    const double pb = p[b];
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    if (i > 0 && (fb || type[b - 1] == T_FLUID)) {
        const int64_t f = ((int64_t)k * ny + j) * (nx + 1) + i;
        u[f] -= dt * (pb - p[b - 1]) / dcx[i];
    }
    if (j > 0 && (fb || type[b - sy] == T_FLUID)) {
        const int64_t f = ((int64_t)k * (ny + 1) + j) * nx + i;
        v[f] -= dt * (pb - p[b - sy]) / dcy[j];
    }
    if (k > 0 && (fb || type[b - sz] == T_FLUID)) {
        const int64_t f = ((int64_t)k * ny + j) * nx + i;
        w[f] -= dt * (pb - p[b - sz]) / dcz[k];
    }
}

hipError_t correct_pass(ibm_grid *g, double *u, double *v, double *w, const double *p, double dt, hipStream_t s) {
    hipLaunchKernelGGL(k_correct, dim3(nblk(g->N)), dim3(256), 0, s, g->type, g->nx, g->ny, g->nz, g->dc0[0], g->dc0[1],
                       g->dc0[2], p, dt, u, v, w);
    return hipGetLastError();
}

// Fractional-step composition (cell-centred momentum, face-normal projection).
// Face velocities from cell-centred components: on every interior face along d the linear
// interpolation between the two centres, (w_b u_a + w_a u_b) / (w_a + w_b) with w the cell
// widths along d; box-wall faces 0 (no flux through the box, as in the convective term).
__global__ void k_cell_to_faces(int nx, int ny, int nz, int d, const double *__restrict__ wd,
                                const double *__restrict__ uc, double *uf) {
    const int fx = nx + (d == 0), fy = ny + (d == 1), fz = nz + (d == 2);
    const int64_t NF = (int64_t)fx * fy * fz;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= NF) return;
    int i, j, k;
    unflatten(id, fx, fy, i, j, k);
    const int q = (d == 0) ? i : (d == 1) ? j : k;
    const int n = (d == 0) ? nx : (d == 1) ? ny : nz;
    if (q == 0 || q == n) {
        uf[id] = 0.0;
        return;
    }
    const int64_t b = ((int64_t)k * ny + j) * nx + i;
    const int64_t a = b - ((d == 0) ? 1 : (d == 1) ? (int64_t)nx : (int64_t)nx * ny);
    const double wa = wd[q - 1], wb = wd[q];
    uf[id] = (wb * uc[a] + wa * uc[b]) / (wa + wb);
}

// Cell-centred correction: on fluid cells u_c -= (delta_{c-1/2} + delta_{c+1/2}) / 2, where
// delta_f = dt (p_b - p_a) / d_f is the correction the projection applies to face f (the
// same arithmetic as k_correct) and 0 on box walls.
__global__ void k_correct_cells(const uint8_t *__restrict__ type, int nx, int ny, int nz, int d,
                                const double *__restrict__ dc, const double *__restrict__ p, double dt, double *uc) {
    const int64_t N = (int64_t)nx * ny * nz;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N || type[id] != T_FLUID) return;
    int i, j, k;
    unflatten(id, nx, ny, i, j, k);
    const int q = (d == 0) ? i : (d == 1) ? j : k;
    const int n = (d == 0) ? nx : (d == 1) ? ny : nz;
    const int64_t st = (d == 0) ? 1 : (d == 1) ? (int64_t)nx : (int64_t)nx * ny;
    const double dm = (q > 0) ? dt * (p[id] - p[id - st]) / dc[q] : 0.0;
    const double dp = (q < n - 1) ? dt * (p[id + st] - p[id]) / dc[q + 1] : 0.0;
    uc[id] -= 0.5 * (dm + dp);
}

hipError_t cell_to_faces_pass(ibm_grid *g, const double *u, const double *v, const double *w, double *uf,
                              double *vf, double *wf, hipStream_t s) {
    const double *c[3] = {u, v, w};
    double *f[3] = {uf, vf, wf};
    for (int d = 0; d < 3; ++d) {
        const int64_t NF = (int64_t)(g->nx + (d == 0)) * (g->ny + (d == 1)) * (g->nz + (d == 2));
        hipLaunchKernelGGL(k_cell_to_faces, dim3(nblk(NF)), dim3(256), 0, s, g->nx, g->ny, g->nz, d, g->w0[d], c[d],
                           f[d]);
    }
    return hipGetLastError();
}

hipError_t correct_cells_pass(ibm_grid *g, double *u, double *v, double *w, const double *p, double dt,
                              hipStream_t s) {
    double *c[3] = {u, v, w};
    for (int d = 0; d < 3; ++d)
        hipLaunchKernelGGL(k_correct_cells, dim3(nblk(g->N)), dim3(256), 0, s, g->type, g->nx, g->ny, g->nz, d,
                           g->dc0[d], p, dt, c[d]);
    return hipGetLastError();
}

__global__ void __launch_bounds__(NORM_NT) k_divmax(Fine<double> F, const double *__restrict__ u,
                                                    const double *__restrict__ v, const double *__restrict__ w,
                                                    double *partials) {
    __shared__ double sh[NORM_NT / 64];
    const int64_t N = (int64_t)F.nx * F.ny * F.nz;
    const int nx = F.nx, ny = F.ny;
    double m = 0.0;
    for (int64_t id = (int64_t)blockIdx.x * NORM_NT + threadIdx.x; id < N; id += (int64_t)gridDim.x * NORM_NT) {
        if (F.type[id] != T_FLUID) continue;
        int i, j, k;
        unflatten(id, nx, ny, i, j, k);
        const int64_t iu = ((int64_t)k * ny + j) * (nx + 1) + i;
        const int64_t iv = ((int64_t)k * (ny + 1) + j) * nx + i;
        const int64_t iw = ((int64_t)k * ny + j) * nx + i;
        double div = (u[iu + 1] - u[iu]) / F.wx[i];
        div = div + (v[iv + nx] - v[iv]) / F.wy[j];
        div = div + (w[iw + (int64_t)nx * ny] - w[iw]) / F.wz[k];
        m = fmax(m, fabs(div));
    }
    double t = block_max<NORM_NT>(m, sh, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ void __launch_bounds__(FIN_NT) k_max_finalize(const double *partials, int nb, double *out) {
    __shared__ double sh[FIN_NT / 64];
    double m = 0.0;
    for (int q = threadIdx.x; q < nb; q += FIN_NT) m = fmax(m, partials[q]);
    m = block_max<FIN_NT>(m, sh, threadIdx.x);
    if (threadIdx.x == 0) *out = m;
}

// max over ghosts of |p_g - sum_m beta_m p_m - h_g| (degenerate ghosts: |p_g - mean of the
// fluid 26-neighbours|), one partial maximum per block
__global__ void __launch_bounds__(256) k_ghost_res(GhostView G, const double *__restrict__ p, int nx, int ny, int nz,
                                                   const uint8_t *__restrict__ type, double *partials) {
    __shared__ double sh[4];
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double r = 0.0;
    if (g < G.ng) {
        const int64_t cell = G.cell[g];
        double target;
        if (G.flags[g] & GF_DEGENERATE) {
            target = fluid_mean26(cell, nx, ny, nz, type, p);
        } else {
            double sm = 0.0;
            for (int m = 0; m < 8; ++m) {
                const int32_t q = G.st[8 * g + m];
                if (q >= 0) sm = sm + G.beta[8 * g + m] * p[q];
            }
            target = sm + G.h[g];
        }
        r = fabs(p[cell] - target);
    }
    r = block_max<256>(r, sh, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = r;
}

hipError_t ghost_residual_pass(ibm_grid *g, const double *p, hipStream_t s) {
    if (g->ng == 0) {
        hipLaunchKernelGGL(k_max_finalize, dim3(1), dim3(FIN_NT), 0, s, g->partials, 0, &g->sc->ghost_res);
        return hipGetLastError();
    }
    const unsigned nb = (unsigned)((g->ng + 255) / 256);
    hipLaunchKernelGGL(k_ghost_res, dim3(nb), dim3(256), 0, s, ghost_view(g), p, g->nx, g->ny, g->nz, g->type,
                       g->partials);
    hipLaunchKernelGGL(k_max_finalize, dim3(1), dim3(FIN_NT), 0, s, g->partials, (int)nb, &g->sc->ghost_res);
    return hipGetLastError();
}

hipError_t divmax_pass(ibm_grid *g, const double *u, const double *v, const double *w, hipStream_t s) {
    hipLaunchKernelGGL(k_divmax, dim3(red_blocks(g->N)), dim3(NORM_NT), 0, s, fine64(g), u, v, w, g->partials);
    hipLaunchKernelGGL(k_max_finalize, dim3(1), dim3(FIN_NT), 0, s, g->partials, red_blocks(g->N), &g->sc->div_max);
    return hipGetLastError();
}

// =======================================================================================
// BiCGStab (paper Section 2.1: the pressure solver family it uses), right-preconditioned by
// one V-cycle, on the fluid + ghost unknowns:
//   A y : fluid rows (S y)_c ; ghost rows s_g (y_g - sum_{m != g} beta_m y_m)
//   b   : fluid rows f       ; ghost rows s_g h_g
// s_g = diagonal of the flux stencil at the ghost cell (both row kinds on one scale).  The
// fluid part of every residual and operator image is projected to zero volume-weighted
// mean (the uniform source shift lambda of the Neumann problem).  All scalars stay on the
// device; the host reads back one status block per iteration.
// =======================================================================================

enum KOp { K_MU = 0, K_ALPHA = 1, K_OMEGA = 2, K_RHO = 3, K_INIT = 4, K_RESTART = 5 };

// ghost scale: the stencil diagonal, summed in the smoother's order
__global__ void k_ghost_scale(int64_t ng, const int32_t *__restrict__ gcell, int nx, int ny, const double *axm,
                              const double *axp, const double *aym, const double *ayp, const double *azm,
                              const double *azp, double *scale) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= ng) return;
    const int64_t id = gcell[g];
    int i, j, k;
    unflatten(id, nx, ny, i, j, k);
    double d = axm[i] + axp[i];
    d = d + aym[j];
    d = d + ayp[j];
    d = d + azm[k];
    d = d + azp[k];
    scale[g] = d;
}

// Ghost rows, before the operator pass (which leaves ghost cells alone): out = s_g (y_g - sum
// beta y) (RESIDUAL: s_g h_g minus that).  Without RESIDUAL also, per block,
// flux: the block's share of the volume-weighted fluid sum of the operator image.  Summed over
//   the fluid rows, V_c (S y)_c = sum_f T_f (y_nb - y_c) cancels on every face between two fluid
//   cells (T_f = V a_f is the same from both sides) and no flux crosses the box walls, so only the
//   faces between a fluid cell c and a ghost cell g remain: sum of V_c a_(c->g) (y_g - y_c).
// gpart[2 block + (0, 1)]: sums of o_g out_g and out_g^2.
// Eight lanes per ghost, one stencil member and one face each, so that a ghost's gathers are in
// flight together: the pass is bound by two round trips.  Flux and rows apart, one thread per
// ghost, the flux added up in a launch between them: 19 us at 128^3, now 4.5 and 2 in the operator.
constexpr int GHOST_ROW_NT = 256, GHOST_ROW_G = GHOST_ROW_NT / 8;
template <bool RESIDUAL>
__global__ void __launch_bounds__(GHOST_ROW_NT)
    k_ghost_rows(GhostView G, Fine<double> F, const double *__restrict__ y, double *out,
                 const double *__restrict__ scale, const double *__restrict__ o, double *flux, double *gpart) {
    const int m = (int)threadIdx.x & 7, nx = F.nx, ny = F.ny, nz = F.nz;
    double acc = 0.0, d0 = 0.0, d1 = 0.0;
    for (int64_t g0 = (int64_t)blockIdx.x * GHOST_ROW_G; g0 < G.ng; g0 += (int64_t)gridDim.x * GHOST_ROW_G) {
        const int64_t g = g0 + (threadIdx.x >> 3);
        const bool live = g < G.ng;
        const int64_t gc = live ? g : 0;
        const int32_t q = G.st[8 * gc + m];
        const double beta = G.beta[8 * gc + m], sc = scale[gc];
        const double h = RESIDUAL ? G.h[gc] : 0.0;
        const int32_t flags = G.flags[gc];
        const int64_t cell = G.cell[gc];
        const double yg = y[cell], og = RESIDUAL ? 0.0 : o[cell];
        double term = live && q >= 0 ? beta * y[max(q, 0)] : 0.0;
        if (!RESIDUAL && live && m < 6) {
            // lanes 0 .. 5: the fluid cell below, above along x, y, z
            const int d = m >> 1, up = m & 1;
            int I[3];
            unflatten(cell, nx, ny, I[0], I[1], I[2]);
            const int at = (d == 0 ? I[0] : d == 1 ? I[1] : I[2]) + (up ? 1 : -1);
            if (at >= 0 && at < (d == 0 ? nx : d == 1 ? ny : nz)) {
                const int64_t step = d == 0 ? 1 : d == 1 ? (int64_t)nx : (int64_t)nx * ny;
                const int64_t c = cell + (up ? step : -step);
                const double *a = up ? (d == 0 ? F.axm : d == 1 ? F.aym : F.azm)
                                     : (d == 0 ? F.axp : d == 1 ? F.ayp : F.azp);
                if (F.type[c] == T_FLUID)
                    acc += ((F.wx[d == 0 ? at : I[0]] * F.wy[d == 1 ? at : I[1]]) * F.wz[d == 2 ? at : I[2]]) * a[at] *
                           (yg - y[c]);
            }
        }
        term += __shfl_xor(term, 1, 64);
        term += __shfl_xor(term, 2, 64);
        term += __shfl_xor(term, 4, 64);
        if (!live || m != 0) continue;
        if (flags & GF_DEGENERATE) term = fluid_mean26(cell, nx, ny, nz, F.type, y);
        const double a = sc * (yg - term);
        const double v = RESIDUAL ? sc * h - a : a;
        out[cell] = v;
        d0 += og * v;
        d1 += v * v;
    }
    if (RESIDUAL) return;
    double sums[3] = {acc, d0, d1};
    __shared__ double sh[GHOST_ROW_NT / 64][3];
    block_sums<GHOST_ROW_NT, 3>(sums, sh, threadIdx.x);
    if (threadIdx.x == 0) flux[blockIdx.x] = sums[0];
    if (threadIdx.x == 1) gpart[2 * blockIdx.x] = sums[1];
    if (threadIdx.x == 2) gpart[2 * blockIdx.x + 1] = sums[2];
}

// The cells in x pairs of the flat order (16-byte accesses, aligned as one element), a contiguous
// range per block; an odd last cell by itself.  The eight streams of k_xr_update at 384^3: 729 us;
// ranges strided over the whole launch 767, single cells 733, x and r in passes of their own 764.
template <typename P, typename L>
__device__ __forceinline__ void for_pairs(const uint8_t *__restrict__ type, int64_t N, P pair, L last) {
    const int64_t step = 2 * (int64_t)blockDim.x, per = (N + step * gridDim.x - 1) / (step * gridDim.x) * step;
    const int64_t end = min(N, per * ((int64_t)blockIdx.x + 1));
    for (int64_t id = per * blockIdx.x + 2 * (int64_t)threadIdx.x; id < end; id += step) {
        if (id + 1 < N) {
            const uint16_t tt = *(const uint16_t *)(type + id);  // type is 256-byte aligned
            pair(id, tt & 0xff, tt >> 8);
        } else {
            last(id, type[id]);
        }
    }
}

// start of the Krylov recurrences on the residual v: projection of its fluid part
// (v -= mu_v; mode 2) or none (restart, mode 3), then rh = v and the sums v.v (all) and v.v
// (fluid).  (The operator images of a step are projected where they are formed.)
__global__ void __launch_bounds__(NORM_NT) k_project(const uint8_t *__restrict__ type, int64_t N, double *v, double *rh,
                                                     const Scalars *sc, int mode, double *partials) {
    const double mu = mode == 3 ? 0.0 : sc->mu_v;
    double s[2] = {0.0, 0.0};
    for_pairs(type, N, [&](int64_t id, int t0, int t1) {
        const DPair x = *(const DPair *)(v + id);
        const DPair r = {t0 == T_FLUID ? x.x - mu : x.x, t1 == T_FLUID ? x.y - mu : x.y};
        if (t0 != T_DEAD && t1 != T_DEAD) {
            if (mode != 3) *(DPair *)(v + id) = r;
            *(DPair *)(rh + id) = r;
        } else {
            if (t0 != T_DEAD) v[id] = rh[id] = r.x;
            if (t1 != T_DEAD) v[id + 1] = rh[id + 1] = r.y;
        }
        const double q0 = t0 == T_DEAD ? 0.0 : r.x * r.x, q1 = t1 == T_DEAD ? 0.0 : r.y * r.y;
        s[0] += q0;
        s[0] += q1;
        s[1] += t0 == T_FLUID ? q0 : 0.0;
        s[1] += t1 == T_FLUID ? q1 : 0.0;
    }, [&](int64_t id, int t) {
        if (t == T_DEAD) return;
        const double r = t == T_FLUID ? v[id] - mu : v[id];
        v[id] = rh[id] = r;
        s[0] += r * r;
        s[1] += t == T_FLUID ? r * r : 0.0;
    });
    block_sums_store<NORM_NT, 2>(s, partials);
}

// Near-breakdown of BiCGStab: an inner product whose modulus is at most brk_tol (the option
// breakdown_tol) times the product of its factors' norms (the shadow residual against the
// residual for rho, or against A y for alpha), or omega = 0.  The step then does not form the
// quotient (alpha = 0; beta = 0) and sets sc->brk; the host restarts the shadow residual from
// the residual.

// NS sums per block: 1 (K_MU), 2 (K_INIT, K_RESTART) or 3 (K_RHO: rh.r, r.r on fluid rows and r.r
// on every active row)
template <int NS>
__global__ void __launch_bounds__(FIN_NT) k_krylov_finalize(const double *partials, int nb, Scalars *sc, int op,
                                                            double brk_tol) {
    double s[NS] = {};
    sum_partials<NS>(partials, nb, s);
    finish_sums<NS>(s);
    if (threadIdx.x != 0) return;
    const double a = s[0], b = s[1 % NS], c = s[2 % NS];
    switch (op) {
        case K_MU: sc->mu_v = a / sc->vol[0]; break;
        case K_RHO:
        case K_INIT:
        case K_RESTART: {
            const double rho_new = a;
            if (op == K_RHO) {
                const bool brk = sc->brk || sc->omega == 0.0 || !(fabs(rho_new) > brk_tol * sqrt(sc->rh2 * c));
                sc->brk = brk ? 1 : 0;
                sc->beta = brk ? 0.0 : (rho_new / sc->rho) * (sc->alpha / sc->omega);
            } else {
                // the shadow residual is (re)started as the residual: rho = rh.rh
                sc->beta = 0.0;
                sc->rh2 = rho_new;
                sc->brk = 0;
            }
            sc->rho_old = sc->rho;
            sc->rho = rho_new;
            sc->norm = sqrt(b);
            sc->rel = (sc->ref > 0.0) ? sc->norm / sc->ref : 0.0;
            if (!isfinite(sc->norm) || !isfinite(sc->beta)) sc->bad = 1;
            if (op == K_INIT) sc->lambda = sc->mu_v;  // the removed mean of b - A x
            break;
        }
    }
}

// alpha = rho / rh.v or omega = t.s / t.t from the operator pass's sums (o w, then w w, of nb
// workgroups) and the ghost rows' (of ngb blocks)
__global__ void __launch_bounds__(FIN_NT) k_krylov_finalize_dots(const double *part, int nb, const double *gpart,
                                                                 int ngb, Scalars *sc, int op, double brk_tol) {
    double s[2] = {0.0, 0.0};
    sum_partials<2>(part, nb, s);
    sum_partials<2>(gpart, ngb, s);
    finish_sums<2>(s);
    if (threadIdx.x != 0) return;
    const double a = s[0], b = s[1];
    if (op == K_ALPHA) {
        // a = rh.v, b = v.v
        if (fabs(a) > brk_tol * sqrt(sc->rh2 * b)) {
            sc->alpha = sc->rho / a;
        } else {
            sc->alpha = 0.0;
            sc->brk = 1;
        }
    } else {
        sc->omega = (b > 0.0) ? a / b : 0.0;
    }
}

// Start of a preconditioner application, by the blocks of the update kernels that take the ghost
// cells: the ghost right-hand sides gh = x_g / s_g of the vector x the kernel forms, and
// e_g = gh (the first ghost refresh of a zero field; 0 at degenerate ghosts, which take the mean
// of their (zero) fluid neighbours).  A pass of its own took 3.6 us, twice a step, for a few
// thousand ghosts.
template <typename T>
struct GhostStart {
    int64_t ng;
    const int32_t *cell, *flags;
    const double *scale;
    double *gh;
    T *e;
    int blocks;  // the first blocks of the launch, one thread per ghost
    __device__ __forceinline__ void put(int64_t g, int64_t id, double x, float *r32) const {
        const double h = x / scale[g];
        gh[g] = h;
        e[id] = (flags[g] & GF_DEGENERATE) ? T(0) : (T)h;
        if (r32) r32[id] = 0.0f;
    }
};

// pd = r + beta (pd - omega v) on fluid + ghost cells
// r32 (mixed precision, else null): the FP32 right-hand side of the preconditioner, the
// fluid part of the result rounded to FP32 and zero elsewhere
// first: the first step of a solve, p = r (beta is 0 and p, v hold nothing yet: not read)
template <typename T>
__global__ void __launch_bounds__(256)
    k_p_update(const uint8_t *__restrict__ type, int64_t N, const double *__restrict__ r, const double *__restrict__ v,
               double *pd, const Scalars *sc, float *r32, int first, GhostStart<T> S) {
    const bool ghosts = (int)blockIdx.x < S.blocks;
    int64_t id = (int64_t)(ghosts ? (int)blockIdx.x : (int)blockIdx.x - S.blocks) * 256 + threadIdx.x;
    if (id >= (ghosts ? S.ng : N)) return;
    const int64_t g = id;
    if (ghosts) id = S.cell[g];
    const uint8_t ty = ghosts ? T_GHOST : type[id];
    if (!ghosts && ty == T_GHOST) return;
    if (ty == T_DEAD) {
        pd[id] = 0.0;
        if (r32) r32[id] = 0.0f;
        return;
    }
    double pv = r[id];
    if (!first) pv = pv + sc->beta * (pd[id] - sc->omega * v[id]);
    __builtin_nontemporal_store(pv, pd + id);
    if (ghosts) S.put(g, id, pv, r32);
    else if (r32) r32[id] = (float)pv;
}

// The BiCGStab vector updates write their full-field results with non-temporal stores (see
// the operator pass).
// s = r - alpha v
template <typename T>
__global__ void __launch_bounds__(256)
    k_s_update(const uint8_t *__restrict__ type, int64_t N, const double *__restrict__ r, const double *__restrict__ v,
               double *s, const Scalars *sc, float *r32, GhostStart<T> S) {
    const bool ghosts = (int)blockIdx.x < S.blocks;
    int64_t id = (int64_t)(ghosts ? (int)blockIdx.x : (int)blockIdx.x - S.blocks) * 256 + threadIdx.x;
    if (id >= (ghosts ? S.ng : N)) return;
    const int64_t g = id;
    if (ghosts) id = S.cell[g];
    const uint8_t ty = ghosts ? T_GHOST : type[id];
    if (!ghosts && ty == T_GHOST) return;
    const double sv = (ty == T_DEAD) ? 0.0 : r[id] - sc->alpha * v[id];
    __builtin_nontemporal_store(sv, s + id);
    if (ghosts) S.put(g, id, sv, r32);
    else if (r32) r32[id] = (ty == T_FLUID) ? (float)sv : 0.0f;
}

// x += alpha y + omega z ; r = s - omega t ; partials of rh.r (all), r.r (fluid) and r.r (all)
__global__ void __launch_bounds__(NORM_NT) k_xr_update(const uint8_t *__restrict__ type, int64_t N, double *x,
                                                       const double *__restrict__ y, const double *__restrict__ z,
                                                       const double *__restrict__ s, const double *__restrict__ t,
                                                       double *r, const double *__restrict__ rh, const Scalars *sc,
                                                       double *partials) {
    const double alpha = sc->alpha, omega = sc->omega;
    double sums[3] = {0.0, 0.0, 0.0};
    auto add = [&](int ty, double rhv, double rv) {
        // selected, not multiplied: the shadow residual is never written on dead cells
        sums[0] += ty == T_DEAD ? 0.0 : rhv * rv;
        sums[1] += ty == T_FLUID ? rv * rv : 0.0;
        sums[2] += ty == T_DEAD ? 0.0 : rv * rv;
    };
    for_pairs(type, N, [&](int64_t id, int t0, int t1) {
        const DPair xv = *(const DPair *)(x + id), yv = *(const DPair *)(y + id), zv = *(const DPair *)(z + id),
                    sv = *(const DPair *)(s + id), tv = *(const DPair *)(t + id), hv = *(const DPair *)(rh + id);
        const DPair xn = {xv.x + alpha * yv.x + omega * zv.x, xv.y + alpha * yv.y + omega * zv.y};
        const DPair rn = {sv.x - omega * tv.x, sv.y - omega * tv.y};
        if (t0 != T_DEAD && t1 != T_DEAD) {
            __builtin_nontemporal_store(xn, (DPair *)(x + id));
            __builtin_nontemporal_store(rn, (DPair *)(r + id));
        } else if (t0 != T_DEAD) {
            x[id] = xn.x;
            r[id] = rn.x;
        } else if (t1 != T_DEAD) {
            x[id + 1] = xn.y;
            r[id + 1] = rn.y;
        }
        add(t0, hv.x, rn.x);
        add(t1, hv.y, rn.y);
    }, [&](int64_t id, int ty) {
        if (ty == T_DEAD) return;
        x[id] = x[id] + alpha * y[id] + omega * z[id];
        const double rv = s[id] - omega * t[id];
        r[id] = rv;
        add(ty, rh[id], rv);
    });
    block_sums_store<NORM_NT, 3>(sums, partials);
}

// The start iterate of a preconditioner application is zero except at the ghost cells, which the
// update kernel before it writes (GhostStart).  k_precond_zero clears both buffers when no
// pre-smoothing sweep comes first; otherwise the start iterate is only read by the first sweep,
// which writes every cell of its output.
template <typename T>
__global__ void k_precond_zero(int64_t N, T *ea, T *eb) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    ea[id] = T(0);
    if (eb) eb[id] = T(0);
}
__global__ void k_widen(const uint8_t *__restrict__ type, int64_t N, const float *__restrict__ e, double *y) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    y[id] = (type[id] == T_DEAD) ? 0.0 : (double)e[id];
}

// whether the next preconditioner application begins with a sweep of the fine level
static bool precond_sweeps(ibm_grid *g, const ibm_solve_opts *o) {
    return o->method == IBM_BICGSTAB_SRJ ? !g->srj_omega.empty() : o->nu1 > 0;
}

// The start iterate of the next preconditioner application (y in ya or yb), cleared if that is
// one of its working buffers; its ghost values are the update kernel's to write (GhostStart).
// begun: that has happened already
template <typename T>
static T *precond_start(ibm_grid *g, double *ya, double *yb, const ibm_solve_opts *o, hipStream_t s, bool begun) {
    const unsigned nbN = (unsigned)nblk(g->N);
    if constexpr (sizeof(T) == 4) {
        if (precond_sweeps(g, o)) return g->pz32;
        if (!begun) hipLaunchKernelGGL(k_precond_zero<float>, dim3(nbN), dim3(256), 0, s, g->N, g->e32a, g->e32b);
        return g->e32a;
    } else {
        if (precond_sweeps(g, o)) return g->pz;
        if (!begun)
            hipLaunchKernelGGL(k_precond_zero<double>, dim3(nbN), dim3(256), 0, s, g->N, ya,
                               o->method == IBM_BICGSTAB_SRJ ? (double *)nullptr : yb);
        return ya;
    }
}

// the first sweep of a preconditioner application (precond_sweeps) and its ghost refresh
template <typename T>
static hipError_t precond_sweep(ibm_grid *g, const double *r, const T *e0, double *yb, const ibm_solve_opts *o,
                                hipStream_t s) {
    hipError_t e;
    T *out;
    if constexpr (sizeof(T) == 4) {
        out = g->e32b;
        e = launch_sweep<float>(FineOf<float>::get(g), e0, out, g->r32, &g->sc->zero32, s);
    } else {
        out = yb;
        if (o->method == IBM_BICGSTAB_SRJ) e = launch_jacobi0(fine64(g), e0, r, out, g->srj_omega[0], s);
        else e = launch_sweep<double>(fine64(g), e0, out, r, &g->sc->zero, s);
    }
    return e != hipSuccess ? e : launch_refresh<T>(g, e0, out, g->g_rhs, s);
}

template <typename T>
static GhostStart<T> ghost_start(ibm_grid *g, T *e) {
    return GhostStart<T>{g->ng, g->g_cell, g->g_flags, g->g_scale, g->g_rhs, e, g->ng > 0 ? (int)nblk(g->ng) : 0};
}

// y = M r: one V-cycle from zero on the error equation with right-hand side r (fluid) and
// ghost right-hand sides r_g / s_g (g->g_rhs, and the start iterate e0 at the ghost cells, both
// written by the kernel that formed r).  FP64: the result lands in one of (ya, yb), returned.
// Mixed: the cycle runs in FP32 on the workspace's FP32 buffers and is widened into ya.
// IBM_BICGSTAB_SRJ: instead of the V-cycle, the scheduled relaxed Jacobi sweeps of the
// grid's schedule, each followed by the ghost refresh (FP64).  swept: precond_sweep is done.
template <typename T>
static hipError_t precondition(ibm_grid *g, const double *r, const T *e0, double *ya, double *yb, double **out,
                               const ibm_solve_opts *o, hipStream_t s, bool swept = false) {
    hipError_t e;
    int cur = swept ? 1 : 0;
    // With pre-smoothing the cycle starts from the start iterate, which the first sweep only
    // reads: no field is cleared per call.
    const T *start = o->nu1 > 0 ? e0 : nullptr;
    if constexpr (sizeof(T) == 4) {
        // g->r32 already holds the FP32 fluid part of r: the update kernel that formed r
        // (k_p_update, k_s_update) wrote it beside r
        float *eb[2] = {g->e32a, g->e32b};
        // with post-smoothing, the last sweep writes the FP64 result itself
        double *wide = o->nu2 > 0 ? ya : nullptr;
        if ((e = vcycle_impl<float>(g, eb, &cur, g->r32, &g->sc->zero32, g->g_rhs, o, s, start, wide, swept)) !=
            hipSuccess)
            return e;
        if (!wide)
            hipLaunchKernelGGL(k_widen, dim3((unsigned)nblk(g->N)), dim3(256), 0, s, g->type, g->N, eb[cur], ya);
        *out = ya;
    } else if (o->method == IBM_BICGSTAB_SRJ) {
        // scheduled relaxed Jacobi: every sweep writes all cells of the other buffer; the first
        // one reads the start iterate (no sweep: the start iterate, in ya, is the result)
        double *bufs[2] = {ya, yb};
        const double *pin = swept ? bufs[cur] : e0;
        const Fine<double> F = fine64(g);
        for (size_t q = swept ? 1 : 0; q < g->srj_omega.size(); ++q) {
            if ((e = launch_jacobi0(F, pin, r, bufs[1 - cur], g->srj_omega[q], s)) != hipSuccess) return e;
            if ((e = launch_refresh<double>(g, pin, bufs[1 - cur], g->g_rhs, s)) != hipSuccess) return e;
            cur = 1 - cur;
            pin = bufs[cur];
        }
        *out = bufs[cur];
    } else {
        double *bufs[2] = {ya, yb};
        if ((e = vcycle_impl<double>(g, bufs, &cur, r, &g->sc->zero, g->g_rhs, o, s, start, nullptr, swept)) !=
            hipSuccess)
            return e;
        *out = bufs[cur];
    }
    return hipGetLastError();
}

// w = P A y (the fluid part with its volume-weighted mean removed) and the inner products of
// `mode` (0: rh.w for alpha; 1: t.s and t.t for omega), then alpha or omega.  The ghost rows come
// first, and with them the mean (from the fluid-ghost faces alone), so the operator pass writes
// the projected image and forms its inner products in the same sweep.
static hipError_t apply_projected(ibm_grid *g, const double *y, double *w, const double *other, int mode, int op,
                                  double brk_tol, hipStream_t s) {
    const int ngb = g->ng > 0 ? std::min(GHOST_ROW_BLOCKS, (int)((g->ng + GHOST_ROW_G - 1) / GHOST_ROW_G)) : 0;
    double *gpart = g->partials + 2 * zmarch_partials_max(g->nx, g->ny, g->nz), *flux = gpart + 2 * GHOST_ROW_BLOCKS;
    if (g->ng > 0)
        hipLaunchKernelGGL(k_ghost_rows<false>, dim3(ngb), dim3(GHOST_ROW_NT), 0, s, ghost_view(g), fine64(g), y, w,
                           g->g_scale, other, flux, gpart);
    int nparts = 0;
    hipError_t e = launch_apply_fluid(fine64(g), y, w, other, MeanParts{flux, ngb, &g->sc->vol[0]}, mode + 1,
                                      g->partials, &nparts, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_krylov_finalize_dots, dim3(1), dim3(FIN_NT), 0, s, g->partials, nparts, gpart, ngb, g->sc, op,
                       brk_tol);
    return hipGetLastError();
}

hipError_t krylov_setup(ibm_grid *g, hipStream_t s) {
    if (g->ng == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ghost_scale, dim3(nblk(g->ng)), dim3(256), 0, s, g->ng, g->g_cell, g->nx, g->ny, g->am0[0],
                       g->ap0[0], g->am0[1], g->ap0[1], g->am0[2], g->ap0[2], g->g_scale);
    return hipGetLastError();
}

// r = P (b - A x), rh = r, rho = rh.r, norm of the fluid part; lambda = removed mean
hipError_t krylov_residual(ibm_grid *g, const double *f, const double *x, hipStream_t s) {
    double *r = g->kv[0], *rh = g->kv[1];
    if (g->ng > 0)
        hipLaunchKernelGGL(k_ghost_rows<true>, dim3((unsigned)((g->ng + GHOST_ROW_G - 1) / GHOST_ROW_G)),
                           dim3(GHOST_ROW_NT), 0, s, ghost_view(g), fine64(g), x, r, g->g_scale, (const double *)nullptr,
                           (double *)nullptr, (double *)nullptr);
    // fluid rows: the z-marching operator pass in its residual form, with sum V r per workgroup
    int nparts = 0;
    hipError_t e = launch_apply_fluid(fine64(g), x, r, f, MeanParts{nullptr, 0, nullptr}, 3, g->partials, &nparts, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_krylov_finalize<1>, dim3(1), dim3(FIN_NT), 0, s, g->partials, nparts, g->sc, (int)K_MU, 0.0);
    const int nb = red_blocks(g->N, 2 * NORM_NT);
    hipLaunchKernelGGL(k_project, dim3(nb), dim3(NORM_NT), 0, s, g->type, g->N, r, rh, g->sc, 2, g->partials);
    hipLaunchKernelGGL(k_krylov_finalize<2>, dim3(1), dim3(FIN_NT), 0, s, g->partials, nb, g->sc, (int)K_INIT, 0.0);
    return hipGetLastError();
}

// The beginning of a BiCGStab step: the new direction, and with AHEAD_SWEEP the first sweep of its
// preconditioner.  It writes the step's scratch vectors alone, so it may be enqueued before the
// host has seen the residual of the step before, and dropped; a restart of the shadow residual
// in between changes nothing either (beta is 0 then: the direction is the residual).
template <typename T>
static hipError_t krylov_ahead_t(ibm_grid *g, const ibm_solve_opts *o, bool first, Ahead what, hipStream_t s) {
    double *r = g->kv[0], *pd = g->kv[2], *v = g->kv[3], *ya = g->kv[6], *yb = g->kv[7];
    float *r32 = sizeof(T) == 4 ? g->r32 : nullptr;  // FP32 right-hand side of the mixed cycle
    T *e0 = precond_start<T>(g, ya, yb, o, s, false);
    const GhostStart<T> S = ghost_start<T>(g, e0);
    hipLaunchKernelGGL(k_p_update<T>, dim3((unsigned)(nblk(g->N) + S.blocks)), dim3(256), 0, s, g->type, g->N, r, v, pd,
                       g->sc, r32, first ? 1 : 0, S);
    if (what == AHEAD_SWEEP && precond_sweeps(g, o)) return precond_sweep<T>(g, pd, e0, yb, o, s);
    return hipGetLastError();
}

hipError_t krylov_ahead(ibm_grid *g, const ibm_solve_opts *o, bool first, Ahead what, hipStream_t s) {
    return o->precision == IBM_MIXED ? krylov_ahead_t<float>(g, o, first, what, s)
                                     : krylov_ahead_t<double>(g, o, first, what, s);
}

// one BiCGStab step on x (kv: r, rh, pd, v, s, t, ya, yb, za, zb), less what was enqueued ahead;
// T: the preconditioner's type
template <typename T>
static hipError_t krylov_step_t(ibm_grid *g, double *x, const ibm_solve_opts *o, bool first, Ahead done,
                                hipStream_t s) {
    double *r = g->kv[0], *rh = g->kv[1], *pd = g->kv[2], *v = g->kv[3], *sv = g->kv[4], *t = g->kv[5];
    double *ya = g->kv[6], *yb = g->kv[7], *za = g->kv[8], *zb = g->kv[9];
    hipError_t e;
    float *r32 = sizeof(T) == 4 ? g->r32 : nullptr;  // FP32 right-hand side of the mixed cycle
    double *y = nullptr, *z = nullptr;
    if (done == AHEAD_NONE && (e = krylov_ahead_t<T>(g, o, first, AHEAD_P, s)) != hipSuccess) return e;
    T *e0 = precond_start<T>(g, ya, yb, o, s, true);
    if ((e = precondition<T>(g, pd, e0, ya, yb, &y, o, s, done == AHEAD_SWEEP && precond_sweeps(g, o))) != hipSuccess)
        return e;
    if ((e = apply_projected(g, y, v, rh, 0, K_ALPHA, o->breakdown_tol, s)) != hipSuccess) return e;
    e0 = precond_start<T>(g, za, zb, o, s, false);
    const GhostStart<T> S = ghost_start<T>(g, e0);
    hipLaunchKernelGGL(k_s_update<T>, dim3((unsigned)(nblk(g->N) + S.blocks)), dim3(256), 0, s, g->type, g->N, r, v, sv,
                       g->sc, r32, S);
    if ((e = precondition<T>(g, sv, e0, za, zb, &z, o, s)) != hipSuccess) return e;
    if ((e = apply_projected(g, z, t, sv, 1, K_OMEGA, o->breakdown_tol, s)) != hipSuccess) return e;
    const int nxr = red_blocks(g->N, 2 * NORM_NT);
    hipLaunchKernelGGL(k_xr_update, dim3(nxr), dim3(NORM_NT), 0, s, g->type, g->N, x, y, z, sv, t, r, rh, g->sc,
                       g->partials);
    hipLaunchKernelGGL(k_krylov_finalize<3>, dim3(1), dim3(FIN_NT), 0, s, g->partials, nxr, g->sc, (int)K_RHO,
                       o->breakdown_tol);
    return hipGetLastError();
}

hipError_t krylov_step(ibm_grid *g, double *x, const ibm_solve_opts *o, bool first, hipStream_t s, Ahead done) {
    return o->precision == IBM_MIXED ? krylov_step_t<float>(g, x, o, first, done, s)
                                     : krylov_step_t<double>(g, x, o, first, done, s);
}

// restart the shadow residual after a breakdown: rh = r, rho = r.r, beta = 0
hipError_t krylov_restart(ibm_grid *g, hipStream_t s) {
    const int nb = red_blocks(g->N, 2 * NORM_NT);
    hipLaunchKernelGGL(k_project, dim3(nb), dim3(NORM_NT), 0, s, g->type, g->N, g->kv[0], g->kv[1], g->sc, 3,
                       g->partials);
    hipLaunchKernelGGL(k_krylov_finalize<2>, dim3(1), dim3(FIN_NT), 0, s, g->partials, nb, g->sc, (int)K_RESTART, 0.0);
    return hipGetLastError();
}

}  // namespace ibm
