// Fused red-black Gauss-Seidel sweep of the coarse multigrid levels that are smoothed level
// by level (Section 2.1: red-black Gauss-Seidel smoothing, applied here to the coarse
// staircase operator of each level).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_util.hpp"
#include "ibm_impl.hpp"

namespace ibm {

// =======================================================================================
// One sweep updates every red cell ((I+J+K) even) from the old values, then every black
// cell from the new red values:
//     e_c = (sum_f T_f e_nb - (R_c - V_c mu)) / sum_f T_f     where sum_f T_f > 0.
// Both colours are done in one out-of-place pass with the z-march of the level-0 sweep: a
// workgroup owns a tile of 64 x BY columns (interior 60 x (BY-4)) and a chunk of planes; at
// step k it forms the red values of plane k+1 and the black values of plane k.  Each thread
// owns two adjacent columns, so it holds one red and one black cell per plane.
// The coarse operator is not separable: each cell carries the transmissibilities of its
// three low faces.  The high faces are the low faces of the +x, +y and +z neighbours: +x
// from the neighbouring lane (a DPP move), +y from LDS, +z from the next plane in the
// queue.  A face is open only when the fine cells on both of its sides are active, so a
// cell with an open face is active and an inactive cell has none: the test sum_f T_f > 0
// already excludes inactive cells, and the activity mask is not read.  Wall faces hold 0.
// Algorithmic traffic per cell: read e, R and three transmissibilities, write e
// (48 B in FP64, 24 B in FP32).
// =======================================================================================

// The compatibility shift of a level's right-hand side, mu = sum of the restriction's partials /
// active volume, formed by the level's first sweep itself (n > 0; every workgroup sums the
// partials, in a fixed order, and the first tile's stores mu for the kernels that follow) instead of by
// a launch of its own, which took 5 us on each level of each cycle.
__device__ __forceinline__ void mu_partial(const MuSource &ms, double *sh) {
    if (threadIdx.x >= 256) return;
    double s = 0.0;
    for (int q = (int)threadIdx.x; q < ms.n; q += 256) s += ms.partials[q];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
}
// after a barrier
__device__ __forceinline__ double mu_total(const MuSource &ms, const double *sh, bool store) {
    const double tot = ((sh[0] + sh[1]) + sh[2]) + sh[3], vol = *ms.vol;
    const double mu = vol > 0.0 ? tot / vol : 0.0;
    if (store && threadIdx.x == 0) *ms.mu = mu;
    return mu;
}

// one plane of a thread's two columns: old values, right-hand side, low-face
// transmissibilities in x, y and z
template <typename T>
struct CPlane {
    using V = typename Pair2<T>::type;
    V e, r, x, y, z;
};

constexpr int SWC_KC_MAX = 512;  // longest z chunk of one workgroup
constexpr int SWC_NC = 64;       // columns of a tile including the 2-column halo
constexpr int SWC_KC_MIN = 8;    // shortest z chunk (each chunk re-reads four planes)
// Levels below this size are swept by bricks (below): there the z-march is bound by the latency
// of its plane steps, not by bandwidth.  With the bricks up to 2^20 cells a wing's FP64 solve
// (levels of 5 x 10^5 and 8 x 10^5) takes 17.0 ms instead of 16.7, a 256^3 mixed one (76^3) 11.22
// instead of 11.42.
template <typename T>
constexpr int64_t SWC_MIN_CELLS = sizeof(T) == 8 ? 3 << 17 : 1 << 20;

// Relaxation value of one cell: the six neighbour products summed from zero in the order
// -x, +x, -y, +y, -z, +z, the diagonal summed in the same order.  A missing neighbour meets
// a zero transmissibility (a wall face, or a high face masked where the level ends), so its
// product is an exact zero; the sum starts at +0 and never becomes -0, so adding that zero
// changes nothing.
template <typename T>
__device__ __forceinline__ T rbc_update(T txm, T txp, T tym, T typ, T tzm, T tzp, T xm, T xp, T ym, T yp, T zm, T zp,
                                        T r, T vol, T mu, T &diag) {
    T s = T(0);
    s = s + txm * xm;
    s = s + txp * xp;
    s = s + tym * ym;
    s = s + typ * yp;
    s = s + tzm * zm;
    s = s + tzp * zp;
    T d = txm + txp;
    d = d + tym;
    d = d + typ;
    d = d + tzm;
    d = d + tzp;
    diag = d;
    return (s - (r - vol * mu)) / d;
}

// Thread layout as in the level-0 sweep: 32 threads span the 64 columns of a tile row; a
// wave holds two rows of the same parity, so the colour phase is uniform per wave and the
// plane loop is specialised for both phases.  VEC (even row length): a thread's column pair
// is 2-element aligned and moves as one access; with an odd row length the two columns are
// loaded and stored one by one.
// Every thread issues the same loads for every plane (addresses clamped into the level);
// values read through clamped addresses are finite copies of level cells that only meet
// zero transmissibilities (walls, or the masked high faces of the last row, column and
// plane), so they enter no result.
// ZERO: the level's correction counts as zero and is not read (a sixth less traffic on a cycle's
// first sweep, and the restriction before it need not clear the field).
template <typename T, int BY, int QD, bool VEC, bool ZERO>
__global__ void __launch_bounds__(32 * BY)
    k_rbgsC_fused(Coarse<T> L, T *__restrict__ eout, MuSource ms, int ntx, int nty, int kc, int ntiles) {
    static_assert(BY % 4 == 0, "two same-parity rows of 32 threads per wave");
    static_assert(QD == 4 || QD == 6, "planes held per thread");
    using V = typename Pair2<T>::type;
    typedef T U2v __attribute__((ext_vector_type(2)));
    typedef U2v U __attribute__((aligned(sizeof(T))));  // a pair at element alignment (odd rows)
    using PD = CPlane<T>;
    constexpr int NC = SWC_NC, TXC = NC - 4, TY = BY - 4;
    __shared__ T so[2][BY][NC + 1];  // old values of the plane whose red values are formed
    __shared__ T sr[2][BY][NC + 1];  // red-updated values of the plane whose black values are formed
    __shared__ T sy[3][BY][NC + 1];  // low-y transmissibilities of the planes, by plane mod 3
    __shared__ T sw[SWC_KC_MAX + 8];  // z widths of planes k0-2 .. k1+5
    const int per = gridDim.x >> 3;
    const int logical = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (logical >= ntiles) return;
    int tile = logical;
    [[maybe_unused]] const int tile0 = tile;
    const int txi = tile % ntx;
    tile /= ntx;
    const int tyi = tile % nty;
    const int chunk = tile / nty;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    const int tx = lane & 31;
    const int ty = (wave >> 1) * 4 + (wave & 1) + 2 * (lane >> 5);
    const int nx = L.n[0], ny = L.n[1], nz = L.n[2];
    const int k0 = chunk * kc, k1 = min(nz, k0 + kc);
    for (int q = (int)threadIdx.x; q < kc + 8; q += 32 * BY) {
        const int kk = k0 - 2 + q;
        sw[q] = (kk >= 0 && kk < nz) ? L.w[2][kk] : T(0);
    }
    const int lc = 2 * tx;
    const int ia = txi * TXC - 2 + lc;  // global column of the first cell (even)
    const int j = tyi * TY - 2 + ty;
    const bool rowin = j >= 0 && j < ny;
    const bool in0 = rowin && ia >= 0 && ia < nx, in1 = rowin && ia + 1 >= 0 && ia + 1 < nx;
    const int yr = min(ty, BY - 1 - ty);
    const int xr0 = min(lc, NC - 1 - lc), xr1 = min(lc + 1, NC - 2 - lc);
    const bool red0 = in0 && yr >= 1 && xr0 >= 1, red1 = in1 && yr >= 1 && xr1 >= 1;
    const bool blk0 = in0 && yr >= 2 && xr0 >= 2, blk1 = in1 && yr >= 2 && xr1 >= 2;
    const bool hx1 = ia + 2 < nx;  // the second cell has a +x neighbour
    const bool hy = j + 1 < ny;    // the row has a +y neighbour
    // element offsets fit 32 bits (a coarse level holds at most 2^28 cells), which lets the
    // loads address from a scalar base plus one 32-bit register
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const int jc = min(max(j, 0), ny - 1);
    const int icv = min(max(ia, 0), nx - 2);
    // Odd row length: rows start at alternating parity, so a thread's pair is only 8-byte
    // aligned; it still moves as one access (the target allows vector accesses at element
    // alignment), starting at icv like the aligned pairs.  On the last column of a row
    // (ia = nx - 1) the pair is (nx - 2, nx - 1) and the thread's first cell is its second
    // element (shifted); its second cell lies past the grid.
    const bool shf = !VEC && ia == nx - 1;
    const uint32_t rowoff = (uint32_t)jc * nx + icv;
    // The outermost halo rows are never updated: their right-hand side and x, z
    // transmissibilities are read from the adjacent row (lines the tile reads anyway), and
    // so is the y transmissibility of the first row (the last row's is the +y face of the
    // row below it).
    const int jr = min(max((ty == 0) ? j + 1 : (ty == BY - 1) ? j - 1 : j, 0), ny - 1);
    const int jy = min(max((ty == 0) ? j + 1 : j, 0), ny - 1);
    const uint32_t roff = (uint32_t)jr * nx + icv, yoff = (uint32_t)jy * nx + icv;
    // unpaired path: the second column is missing at the high wall of an odd row, where the
    // first column's high face is the wall (its x transmissibility must read 0, not the
    // clamped copy of the first column's low face)
    const bool x1in = VEC || ia + 1 < nx;
    const T vxy0 = in0 ? L.w[0][ia] * L.w[1][jc] : T(0);
    const T vxy1 = in1 ? L.w[0][ia + 1] * L.w[1][jc] : T(0);
    __shared__ double smu[4];
    if (ms.n > 0) {
        mu_partial(ms, smu);
        __syncthreads();
    }
    const T mu = ms.n > 0 ? (T)mu_total(ms, smu, tile0 == 0) : (T)(*L.mu);
    // LDS rows and columns of the neighbours, clamped into the tile (lanes whose result is
    // discarded read valid entries)
    const int rym = max(ty - 1, 0), ryp = min(ty + 1, BY - 1);
    const int cm0 = max(lc - 1, 0), cp1 = min(lc + 2, NC - 1);
    const bool phase = ((wave + (tyi * TY) + k0) & 1) != 0;
    const int klast = min(k1 + 1, nz - 1);
    const T *__restrict__ pe = L.e;
    const T *__restrict__ pr = L.R;
    const T *__restrict__ px = L.Tl[0];
    const T *__restrict__ py = L.Tl[1];
    const T *__restrict__ pz = L.Tl[2];
    auto load = [=](int k) -> PD {
        PD d;
        const uint32_t base = (uint32_t)min(max(k, 0), klast) * plane;
        if constexpr (VEC) {
            d.e = ZERO ? V{T(0), T(0)} : *reinterpret_cast<const V *>(pe + base + rowoff);
            d.r = *reinterpret_cast<const V *>(pr + base + roff);
            d.x = *reinterpret_cast<const V *>(px + base + roff);
            d.y = *reinterpret_cast<const V *>(py + base + yoff);
            d.z = *reinterpret_cast<const V *>(pz + base + roff);
        } else {
            const U e2 = ZERO ? U{T(0), T(0)} : *reinterpret_cast<const U *>(pe + base + rowoff);
            const U r2 = *reinterpret_cast<const U *>(pr + base + roff);
            const U x2 = *reinterpret_cast<const U *>(px + base + roff);
            const U y2 = *reinterpret_cast<const U *>(py + base + yoff);
            const U z2 = *reinterpret_cast<const U *>(pz + base + roff);
            d.e.x = shf ? e2.y : e2.x;
            d.e.y = e2.y;
            d.r.x = shf ? r2.y : r2.x;
            d.r.y = r2.y;
            d.x.x = shf ? x2.y : x2.x;
            d.x.y = x1in ? x2.y : T(0);
            d.y.x = shf ? y2.y : y2.x;
            d.y.y = y2.y;
            d.z.x = shf ? z2.y : z2.x;
            d.z.y = z2.y;
        }
        return d;
    };
    // LDS buffer of plane q's y transmissibilities (q >= k0 - 1)
#define IBMC_YB(q) (((q) - k0 + 3) % 3)

    // Red-updated values of plane q from M = plane q-1, C = plane q, P = plane q+1, OB = LDS
    // of the old values of plane q.  FR (compile-time): the first cell is the red one.
#define IBMC_RED(q, M, C, P, OB, R0, R1, FR)                                                                       \
    {                                                                                                              \
        const int l_ = (FR) ? lc : lc + 1;                                                                         \
        const T xn_ = lane_above((C).x.x);                                                                         \
        const T txm_ = (FR) ? (C).x.x : (C).x.y;                                                                   \
        const T txp_ = (FR) ? (C).x.y : (hx1 ? xn_ : T(0));                                                        \
        const T tym_ = (FR) ? (C).y.x : (C).y.y;                                                                   \
        const T typ_ = hy ? sy[IBMC_YB(q)][ryp][l_] : T(0);                                                        \
        const T tzm_ = (FR) ? (C).z.x : (C).z.y;                                                                   \
        const T tzp_ = ((q) + 1 < nz) ? ((FR) ? (P).z.x : (P).z.y) : T(0);                                         \
        T d_;                                                                                                      \
        const T v_ = rbc_update<T>(txm_, txp_, tym_, typ_, tzm_, tzp_, OB[ty][(FR) ? cm0 : lc], OB[ty][(FR) ? lc + 1 : cp1], \
                                   OB[rym][l_], OB[ryp][l_], (FR) ? (M).e.x : (M).e.y, (FR) ? (P).e.x : (P).e.y,    \
                                   (FR) ? (C).r.x : (C).r.y, ((FR) ? vxy0 : vxy1) * sw[(q) - k0 + 2], mu, d_);      \
        const bool live_ = ((FR) ? red0 : red1) && (q) >= 0 && (q) < nz && d_ > T(0);                             \
        R0 = ((FR) && live_) ? v_ : (C).e.x;                                                                       \
        R1 = (!(FR) && live_) ? v_ : (C).e.y;                                                                      \
    }

    // One plane step: A = plane k, B = k+1, C = k+2 (QD - 3 more planes in flight);
    // afterwards the slot A receives plane k + QD.  Steps past the chunk end compute from clamped data
    // and store nothing.  The lanes meet again after the store: without that, and with ZERO's values
    // known, the compiler made the store's branch the end of an inner loop over the plane steps, in
    // which the lanes that store nothing (the halo) went on through barriers and lane moves of later
    // steps while the others were switched off, and even rows came out wrong by 1e-3.
#define IBMC_STEP(A, B, C, k, FR)                                                                                  \
    {                                                                                                              \
        so[buf][ty][lc] = (B).e.x;                                                                                 \
        so[buf][ty][lc + 1] = (B).e.y;                                                                             \
        sr[buf][ty][lc] = pb0;                                                                                     \
        sr[buf][ty][lc + 1] = pb1;                                                                                 \
        sy[IBMC_YB((k) + 1)][ty][lc] = (B).y.x;                                                                    \
        sy[IBMC_YB((k) + 1)][ty][lc + 1] = (B).y.y;                                                                \
        __syncthreads();                                                                                           \
        T pc0, pc1;                                                                                                \
        IBMC_RED((k) + 1, A, B, C, so[buf], pc0, pc1, FR);                                                         \
        T out0, out1;                                                                                              \
        {                                                                                                          \
            const int l_ = (FR) ? lc : lc + 1;                                                                     \
            const T xn_ = lane_above((A).x.x);                                                                     \
            const T txm_ = (FR) ? (A).x.x : (A).x.y;                                                               \
            const T txp_ = (FR) ? (A).x.y : (hx1 ? xn_ : T(0));                                                    \
            const T tym_ = (FR) ? (A).y.x : (A).y.y;                                                               \
            const T typ_ = hy ? sy[IBMC_YB(k)][ryp][l_] : T(0);                                                    \
            const T tzm_ = (FR) ? (A).z.x : (A).z.y;                                                               \
            const T tzp_ = ((k) + 1 < nz) ? ((FR) ? (B).z.x : (B).z.y) : T(0);                                     \
            T d_;                                                                                                  \
            const T v_ = rbc_update<T>(txm_, txp_, tym_, typ_, tzm_, tzp_, sr[buf][ty][(FR) ? cm0 : lc],           \
                                       sr[buf][ty][(FR) ? lc + 1 : cp1], sr[buf][rym][l_], sr[buf][ryp][l_],       \
                                       (FR) ? pa0 : pa1, (FR) ? pc0 : pc1, (FR) ? (A).r.x : (A).r.y,               \
                                       ((FR) ? vxy0 : vxy1) * sw[(k) - k0 + 2], mu, d_);                           \
            const bool live_ = ((FR) ? blk0 : blk1) && d_ > T(0);                                                  \
            out0 = ((FR) && live_) ? v_ : pb0;                                                                     \
            out1 = (!(FR) && live_) ? v_ : pb1;                                                                    \
        }                                                                                                          \
        if constexpr (VEC) {                                                                                       \
            if ((k) < k1 && blk0) { /* a pair is wholly inside or outside the tile interior */                    \
                V o_;                                                                                              \
                o_.x = out0;                                                                                       \
                o_.y = out1;                                                                                       \
                *reinterpret_cast<V *>(eout + ((uint32_t)(k) * plane + (uint32_t)j * nx + ia)) = o_;                   \
            }                                                                                                      \
        } else if ((k) < k1) { /* both cells or, at the last column of a row, the first alone */                  \
            const uint32_t o_ = (uint32_t)(k) * plane + (uint32_t)j * nx + ia;                                     \
            if (blk0 && blk1) {                                                                                    \
                U o2_;                                                                                             \
                o2_.x = out0;                                                                                      \
                o2_.y = out1;                                                                                      \
                *reinterpret_cast<U *>(eout + o_) = o2_;                                                           \
            } else if (blk0) {                                                                                     \
                eout[o_] = out0;                                                                                   \
            }                                                                                                      \
        }                                                                                                          \
        pa0 = pb0;                                                                                                 \
        pa1 = pb1;                                                                                                 \
        pb0 = pc0;                                                                                                 \
        pb1 = pc1;                                                                                                 \
        buf ^= 1;                                                                                                  \
        __builtin_amdgcn_wave_barrier();                                                                           \
        A = load((k) + QD);                                                                                        \
    }

    // Queue of QD planes: at step k the slots hold planes k .. k+QD-1 (the last QD-3 in
    // flight); unrolled by the queue depth so the slots change roles by name and no in-flight
    // load is ever copied.  S: the first cell is red at plane k0 - 1.
#define IBMC_BODY(S)                                                                                               \
    {                                                                                                              \
        PD q0 = load(k0 - 2), q1 = load(k0 - 1), q2 = load(k0), q3 = load(k0 + 1);                                 \
        [[maybe_unused]] PD q4, q5;                                                                                \
        if constexpr (QD == 6) {                                                                                   \
            q4 = load(k0 + 2);                                                                                     \
            q5 = load(k0 + 3);                                                                                     \
        }                                                                                                          \
        T pa0, pa1, pb0, pb1;                                                                                      \
        so[0][ty][lc] = q1.e.x;                                                                                    \
        so[0][ty][lc + 1] = q1.e.y;                                                                                \
        sy[IBMC_YB(k0 - 1)][ty][lc] = q1.y.x;                                                                      \
        sy[IBMC_YB(k0 - 1)][ty][lc + 1] = q1.y.y;                                                                  \
        sy[IBMC_YB(k0)][ty][lc] = q2.y.x;                                                                          \
        sy[IBMC_YB(k0)][ty][lc + 1] = q2.y.y;                                                                      \
        __syncthreads();                                                                                           \
        IBMC_RED(k0 - 1, q0, q1, q2, so[0], pa0, pa1, (S));                                                        \
        q0 = load(k0 + QD - 2);                                                                                    \
        so[1][ty][lc] = q2.e.x;                                                                                    \
        so[1][ty][lc + 1] = q2.e.y;                                                                                \
        __syncthreads();                                                                                           \
        IBMC_RED(k0, q1, q2, q3, so[1], pb0, pb1, !(S));                                                           \
        q1 = load(k0 + QD - 1);                                                                                    \
        int buf = 0;                                                                                               \
        if constexpr (QD == 4) {                                                                                   \
            for (int k = k0; k < k1; k += 4) {                                                                     \
                IBMC_STEP(q2, q3, q0, k, (S));                                                                     \
                IBMC_STEP(q3, q0, q1, k + 1, !(S));                                                                \
                IBMC_STEP(q0, q1, q2, k + 2, (S));                                                                 \
                IBMC_STEP(q1, q2, q3, k + 3, !(S));                                                                \
            }                                                                                                      \
        } else {                                                                                                   \
            for (int k = k0; k < k1; k += 6) {                                                                     \
                IBMC_STEP(q2, q3, q4, k, (S));                                                                     \
                IBMC_STEP(q3, q4, q5, k + 1, !(S));                                                                \
                IBMC_STEP(q4, q5, q0, k + 2, (S));                                                                 \
                IBMC_STEP(q5, q0, q1, k + 3, !(S));                                                                \
                IBMC_STEP(q0, q1, q2, k + 4, (S));                                                                 \
                IBMC_STEP(q1, q2, q3, k + 5, !(S));                                                                \
            }                                                                                                      \
        }                                                                                                          \
    }

    if (phase) IBMC_BODY(true) else IBMC_BODY(false)
#undef IBMC_BODY
#undef IBMC_STEP
#undef IBMC_RED
#undef IBMC_YB
}

// Tile rows and queue depth per precision.  FP64: 16 rows (512 threads, so the plane queue
// stays in registers; 32 rows spill it) and four planes (a deeper queue measured slower).
// FP32: 32 rows, four planes.
template <typename T>
struct SwcRows;
template <>
struct SwcRows<double> {
    static constexpr int BY = 16, QD = 4;
};
template <>
struct SwcRows<float> {
    static constexpr int BY = 32, QD = 4;
};

// Bricks hold SWB_Y x SWB_Z rows of up to SWB_COLS columns.
constexpr int SWB_Y = 4, SWB_Z = 4, SWB_W = 8, SWB_COLS = 64;
static int sweepC_brick_tiles(int nx) {  // one tile needs no halo
    return nx <= SWB_COLS ? 1 : (nx + SWB_COLS - 5) / (SWB_COLS - 4);
}

// Levels whose bricks are a quarter full at most (16 columns, or one plane), where there are many
// bricks: a brick's cost does not depend on how full it is.  Such levels take a launch per colour or,
// from 393k cells, the z-march.  Us that bricks on all of a grid's levels add to a V(2,2) cycle with
// those: 3 x 360 x 360 (level 1 of 2025 bricks) 531 + 68, 3 x 512 x 512 (4096) 840 + 147,
// 2 x 40000 x 1 (5000) 388 + 304, 1500^2 in FP32 (2444) 371 + 29, 512^2 (1152) 181 + 1, 559^2 (1400) 355 - 23.
static bool sweepC_narrow(const int n[3]) {
    const int64_t bricks =
        (int64_t)sweepC_brick_tiles(n[0]) * ((n[1] + SWB_Y - 1) / SWB_Y) * ((n[2] + SWB_Z - 1) / SWB_Z);
    return bricks > 1536 && (int64_t)n[0] * n[1] * n[2] <= 256 * bricks;
}

// The sweep of a smaller level by bricks: the scheme of the fine level's bricks (sweepb.hip) with
// the coarse operator.  Half a wave takes a row of 64 columns, a lane two adjacent columns; each
// of the NT row takers updates NI rows of the brick's BY x BZ and NH of the ring around them, and
// loads right-hand sides and transmissibilities of its rows along with the old values, all in
// flight together.  zero: the level's correction is still zero, so no old values are read.
// Two launches of one colour each took 2 x 4.7 us on levels of 10^4 to 10^5 cells; one of these
// takes 5.9 to 6.3 us there (FP64) and 12.4 us at 72^3.  Cell by cell the operations are those of rbc_update, and a cell
// without an open face keeps its value.
template <typename T, int BY, int BZ, int NW>
__global__ void __launch_bounds__(64 * NW, 4)
    k_rbgsC_brick(Coarse<T> L, T *__restrict__ eout, MuSource ms, int zero, int ntx, int nty, int bx, int xoff,
                  int ntiles) {
    constexpr int LW = 32, NT = 2 * NW;
    constexpr int HY = BY + 4, HZ = BZ + 4, ROWS = HY * HZ, NL = (ROWS + NT - 1) / NT;
    constexpr int SIDES = 2 * (BZ + 2), RING = SIDES + 2 * BY;
    constexpr int NI = BY * BZ / NT, NH = (RING + NT - 1) / NT, NU = NI + NH;
    static_assert(NI * NT == BY * BZ, "interior rows divide among the takers");
    typedef T U2 __attribute__((ext_vector_type(2)));
    typedef U2 U __attribute__((aligned(sizeof(T))));
    constexpr int P = LW + 1;
    __shared__ T s[2][ROWS][P];  // even and odd columns, with guards: see sweepb.hip
    __shared__ double smu[4];
    const int per = gridDim.x >> 3;
    const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (tile >= ntiles) return;
    const int nx = L.n[0], ny = L.n[1], nz = L.n[2], tid = (int)threadIdx.x;
    const int l = tid & (LW - 1), me = tid / LW;
    const int x0 = tile % ntx * bx - xoff, y0 = tile / ntx % nty * BY - 2, z0 = tile / (ntx * nty) * BZ - 2;
    const int i = x0 + 2 * l;
    const bool in0 = i >= 0 && i < nx, in1 = i >= 0 && i + 1 < nx, in2 = i >= 0 && i + 2 < nx;
    // unconditional loads at clamped places; what lies outside meets zero transmissibilities
    const uint32_t ic = (uint32_t)min(max(i, 0), nx - 2), ip = (uint32_t)min(max(i + 2, 0), nx - 1);
    const bool shf = i == nx - 1;
    auto cell = [&](int y, int z) -> uint32_t {  // a level below SWC_MIN_CELLS: 24 bits
        const uint32_t j = (uint32_t)min(max(y0 + y, 0), ny - 1), k = (uint32_t)min(max(z0 + z, 0), nz - 1);
        return __umul24(__umul24(k, (uint32_t)ny) + j, (uint32_t)nx);
    };
    auto pair = [&](const T *a, uint32_t c) -> U {
        U v = *reinterpret_cast<const U *>(a + c);
        if (shf) v.x = v.y;
        return v;
    };
    U v[NL];
    {
        int y = me % HY, z = me / HY;
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            v[q] = U{T(0), T(0)};
            if (!zero) v[q] = pair(L.e, cell(y, z) + ic);
            y += NT % HY;
            z += NT / HY;
            if (y >= HY) {
                y -= HY;
                ++z;
            }
        }
    }
    // the rows this taker updates.  Interior rows need both cells of the pair, ring rows the red one.
    int yu[NU], zu[NU];
    bool row[NU];
    U r[NI], tx[NI], ty[NI], tyh[NI], tz[NI], tzh[NI];
    T txh[NI], g[NH][7];
#pragma unroll
    for (int q = 0; q < NU; ++q) {
        bool any = true;
        if (q < NI) {
            const int e = q * NT + me;
            yu[q] = e % BY + 2;
            zu[q] = e / BY + 2;
        } else {
            const int e = (q - NI) * NT + me, u = e - SIDES;
            any = e < RING;
            yu[q] = !any ? 1 : e < SIDES ? ((e & 1) ? BY + 2 : 1) : u % BY + 2;
            zu[q] = !any ? 1 : e < SIDES ? (e >> 1) + 1 : u / BY ? BZ + 2 : 1;
        }
        const int j = y0 + yu[q], k = z0 + zu[q];
        row[q] = any && j >= 0 && j < ny && k >= 0 && k < nz;
        const uint32_t c0 = cell(yu[q], zu[q]), cy = cell(yu[q] + 1, zu[q]), cz = cell(yu[q], zu[q] + 1);
        const bool hy = j + 1 < ny, hz = k + 1 < nz;
        if (q < NI) {
            r[q] = pair(L.R, c0 + ic);
            tx[q] = pair(L.Tl[0], c0 + ic);
            txh[q] = L.Tl[0][c0 + ip];
            ty[q] = pair(L.Tl[1], c0 + ic);
            tyh[q] = pair(L.Tl[1], cy + ic);
            tz[q] = pair(L.Tl[2], c0 + ic);
            tzh[q] = pair(L.Tl[2], cz + ic);
            if (!in1) tx[q].y = T(0);  // the first cell's high face is the wall
            if (!in2) txh[q] = T(0);
            if (!hy) tyh[q] = U{T(0), T(0)};
            if (!hz) tzh[q] = U{T(0), T(0)};
        } else {
            const int x = i + ((j + k) & 1);
            const uint32_t xc = (uint32_t)min(max(x, 0), nx - 1), xp = (uint32_t)min(max(x + 1, 0), nx - 1);
            T(&h)[7] = g[q - NI];
            h[0] = L.Tl[0][c0 + xc];
            h[1] = L.Tl[0][c0 + xp];
            h[2] = L.Tl[1][c0 + xc];
            h[3] = L.Tl[1][cy + xc];
            h[4] = L.Tl[2][c0 + xc];
            h[5] = L.Tl[2][cz + xc];
            h[6] = L.R[c0 + xc];
            if (x + 1 >= nx) h[1] = T(0);
            if (!hy) h[3] = T(0);
            if (!hz) h[5] = T(0);
        }
    }
    const T wx[2] = {in0 ? L.w[0][i] : T(0), in1 ? L.w[0][i + 1] : T(0)};
    if (ms.n > 0) mu_partial(ms, smu);
    for (int q = tid; q < ROWS; q += 64 * NW) s[1][q][0] = s[0][q][LW] = T(0);
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int rr = q * NT + me;
        if (rr < ROWS) {
            s[0][rr][l] = v[q].x;
            s[1][rr][l + 1] = v[q].y;
        }
    }
    __syncthreads();
    const T mu = ms.n > 0 ? (T)mu_total(ms, smu, tile == 0) : (T)(*L.mu);
    // the cell of parity b of the pair in the taker's row q; live: it has an open face
    auto update = [&](int q, int b, T &own, bool &live) -> T {
        const T *p = &s[0][zu[q] * HY + yu[q]][l];
        const T *c = p + (b ? ROWS * P + 1 : 0), *o = p + (b ? 0 : ROWS * P + 1);
        own = o[0];
        const T side = o[b ? 1 : -1];
        const int j = min(max(y0 + yu[q], 0), ny - 1), k = min(max(z0 + zu[q], 0), nz - 1);
        const T vol = ((b ? wx[1] : wx[0]) * L.w[1][j]) * L.w[2][k];
        T d, n;
        if (q < NI) {
            n = rbc_update<T>(b ? tx[q].y : tx[q].x, b ? txh[q] : tx[q].y, b ? ty[q].y : ty[q].x,
                              b ? tyh[q].y : tyh[q].x, b ? tz[q].y : tz[q].x, b ? tzh[q].y : tzh[q].x,
                              b ? own : side, b ? side : own, c[-P], c[P], c[-P * HY], c[P * HY],
                              b ? r[q].y : r[q].x, vol, mu, d);
        } else {
            const T(&h)[7] = g[q - NI];
            n = rbc_update<T>(h[0], h[1], h[2], h[3], h[4], h[5], b ? own : side, b ? side : own, c[-P], c[P],
                              c[-P * HY], c[P * HY], h[6], vol, mu, d);
        }
        live = row[q] && (b ? in1 : in0) && d > T(0);
        return n;
    };
    T own;
    bool live;
#pragma unroll
    for (int q = 0; q < NU; ++q) {
        const int b = (y0 + yu[q] + z0 + zu[q]) & 1;  // x0 is even
        const T n = update(q, b, own, live);
        if (live) s[b][zu[q] * HY + yu[q]][l + b] = n;
    }
    __syncthreads();
    const bool mine = 2 * l >= xoff && 2 * l < xoff + bx && in0;
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        const int b = (y0 + yu[q] + z0 + zu[q] + 1) & 1;
        const T n = update(q, b, own, live);
        const T x = live ? n : s[b][zu[q] * HY + yu[q]][l + b];
        T *o = eout + cell(yu[q], zu[q]) + i;
        const U pr = U{b ? own : x, b ? x : own};
        if (mine && row[q] && in1) *reinterpret_cast<U *>(o) = pr;
        else if (mine && row[q]) *o = pr.x;
    }
}

// One colour of a sweep, in place: a thread per cell of that colour (in each x pair of a row exactly
// one cell has it), every load issued before the test.  For levels of many short rows.
template <typename T>
__global__ void k_sweepC(Coarse<T> L, int colour) {
    const int nx = L.n[0], ny = L.n[1], nz = L.n[2], hx = (nx + 1) >> 1;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)hx * ny * nz) return;
    int P, J, K;
    unflatten(t, hx, ny, P, J, K);
    const int I = 2 * P + ((J + K + colour) & 1);
    if (I >= nx) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny, id = (int64_t)K * sz + (int64_t)J * sy + I;
    // places clamped into the level: a neighbour beyond a wall meets a zero transmissibility
    const int64_t xm = id - (I > 0), xp = id + (I < nx - 1), ym = id - (J > 0 ? sy : 0), yp = id + (J < ny - 1 ? sy : 0),
                  zm = id - (K > 0 ? sz : 0), zp = id + (K < nz - 1 ? sz : 0);
    const T *Tx = L.Tl[0], *Ty = L.Tl[1], *Tz = L.Tl[2];
    const T txp = I < nx - 1 ? Tx[xp] : T(0), typ = J < ny - 1 ? Ty[yp] : T(0), tzp = K < nz - 1 ? Tz[zp] : T(0);
    const T vol = (L.w[0][I] * L.w[1][J]) * L.w[2][K];
    T d;
    const T v = rbc_update<T>(Tx[id], txp, Ty[id], typ, Tz[id], tzp, L.e[xm], L.e[xp], L.e[ym], L.e[yp], L.e[zm],
                              L.e[zp], L.R[id], vol, (T)(*L.mu), d);
    if (d > T(0)) L.e[id] = v;
}

bool sweepC_by_colours(const int n[3]) {
    return sweepC_narrow(n) && (int64_t)n[0] * n[1] * n[2] < SWC_MIN_CELLS<double>;
}

template <typename T>
hipError_t launch_sweepC_colours(const Coarse<T> &L, hipStream_t s) {
    const int64_t np = (int64_t)((L.n[0] + 1) / 2) * L.n[1] * L.n[2];
    for (int colour = 0; colour < 2; ++colour)
        hipLaunchKernelGGL(k_sweepC<T>, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, L, colour);
    return hipGetLastError();
}

// Launch of a sweep: bricks, or the z-march in chunks of kc planes; rounds of workgroups that run at once
struct SweepCTiles {
    bool bricks;
    int ntx, nty, kc, ntiles;
    int64_t rounds;
};
template <typename T>
static SweepCTiles sweepC_tiles(const int n[3]) {
    SweepCTiles t;
    t.bricks = (int64_t)n[0] * n[1] * n[2] < SWC_MIN_CELLS<T> && !sweepC_narrow(n);
    const int slots = device_cu_count();
    if (t.bricks) {
        t.ntx = sweepC_brick_tiles(n[0]);
        t.nty = (n[1] + SWB_Y - 1) / SWB_Y;
        t.kc = SWB_Z;
        t.ntiles = t.ntx * t.nty * ((n[2] + SWB_Z - 1) / SWB_Z);
        t.rounds = (t.ntiles + 2 * slots - 1) / (2 * slots);  // two of 512 threads at its register count
        return t;
    }
    constexpr int TXC = SWC_NC - 4, TY = SwcRows<T>::BY - 4;
    t.ntx = (n[0] + TXC - 1) / TXC;
    t.nty = (n[1] + TY - 1) / TY;
    const int64_t per_slab = (int64_t)t.ntx * t.nty;
    // one workgroup per CU; chunks as long as that residency allows, but no shorter than
    // kcmin planes (each chunk re-reads four planes of its neighbours)
    const int kcmin = SWC_KC_MIN;
    int nchunk = (int)std::max<int64_t>(1, std::min<int64_t>(slots / per_slab, n[2]));
    int kc = (n[2] + nchunk - 1) / nchunk;
    kc = std::max(kc, std::min(kcmin, n[2]));
    kc = std::min(kc, SWC_KC_MAX);
    nchunk = (n[2] + kc - 1) / kc;
    t.kc = kc;
    t.ntiles = (int)(per_slab * nchunk);
    t.rounds = (t.ntiles + slots - 1) / slots;
    return t;
}

// Every workgroup sums all partials, about 17 us for 65536 of them, one round of workgroups after the
// other; a launch that sums them once takes 5 us and 12 us for 32768.  On levels of 2048^2 cells (32768
// partials, 24 rounds) the first sweep took 282 us instead of 87.
template <typename T>
bool sweepC_forms_mu(const int n[3], int nparts) {
    return sweepC_tiles<T>(n).rounds * nparts <= 24576;
}

template <typename T>
hipError_t launch_sweepC(const Coarse<T> &L, T *eout, const MuSource &ms, bool zero, hipStream_t s) {
    if (L.n[0] < 2) return hipErrorInvalidValue;
    const SweepCTiles t = sweepC_tiles<T>(L.n);
    const int grid = (t.ntiles + 7) / 8 * 8;
    if (t.bricks) {
        const int xoff = t.ntx == 1 ? 0 : 2, bx = t.ntx == 1 ? SWB_COLS : (((L.n[0] + t.ntx - 1) / t.ntx + 1) & ~1);
        hipLaunchKernelGGL((k_rbgsC_brick<T, SWB_Y, SWB_Z, SWB_W>), dim3(grid), dim3(64 * SWB_W), 0, s, L, eout, ms,
                           zero ? 1 : 0, t.ntx, t.nty, bx, xoff, t.ntiles);
        return hipGetLastError();
    }
    constexpr int BY = SwcRows<T>::BY, QD = SwcRows<T>::QD;
    const bool vec = (L.n[0] & 1) == 0;
    auto k = vec ? (zero ? k_rbgsC_fused<T, BY, QD, true, true> : k_rbgsC_fused<T, BY, QD, true, false>)
                 : (zero ? k_rbgsC_fused<T, BY, QD, false, true> : k_rbgsC_fused<T, BY, QD, false, false>);
    hipLaunchKernelGGL(k, dim3(grid), dim3(32 * BY), 0, s, L, eout, ms, t.ntx, t.nty, t.kc, t.ntiles);
    return hipGetLastError();
}

template bool sweepC_forms_mu<double>(const int[3], int);
template bool sweepC_forms_mu<float>(const int[3], int);
template hipError_t launch_sweepC<double>(const Coarse<double> &, double *, const MuSource &, bool, hipStream_t);
template hipError_t launch_sweepC<float>(const Coarse<float> &, float *, const MuSource &, bool, hipStream_t);
template hipError_t launch_sweepC_colours<double>(const Coarse<double> &, hipStream_t);
template hipError_t launch_sweepC_colours<float>(const Coarse<float> &, hipStream_t);

}  // namespace ibm
