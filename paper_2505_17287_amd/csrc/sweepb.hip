// Red-black Gauss-Seidel sweep of the fine level by bricks, for grids too small for the z-march
// of sweep.hip (paper Section 2.1: red-black Gauss-Seidel smoothing).
//
// The z-march holds one plane of 64 x 32 columns per step and one barrier per plane; below a few
// million cells its tiles leave compute units idle and the serial plane steps set the time
// (128^3: 120 workgroups of 20 steps, 26 us for 52 MB).  Here a workgroup takes a brick: it loads
// the old values with a halo of two cells, all loads in flight together, into LDS and keeps its
// own rows in registers too, updates the red cells of the brick and of one halo layer, then the
// black cells of the brick, and stores the brick.  Two barriers in all.  The halo is re-read from
// L2 and its red cells are recomputed, which costs bandwidth and issue slots: the z-march stays
// better where both are the limit (by_bricks has the sizes).
// Cell by cell the operations and their order are those of the two-pass definition, so the
// result is bitwise that of the z-march.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "ibm_impl.hpp"

namespace ibm {

// A half or whole wave takes a row (x line) at a time, a lane two adjacent columns (the first
// even): RPW rows per wave, each of 128 / RPW columns: bx of the brick and the halo (xoff columns
// on the left).  The rows to update are dealt out with the NI interior ones of each taker first,
// then its NH of the ring around them, so that every loop is branch-free and unrolled and the
// LDS round trips of several rows overlap.  BZ = 1: a grid of one plane, without a z halo.
template <typename T, typename TO, int RPW, int BY, int BZ, int NW>
__global__ void __launch_bounds__(64 * NW, 4)
    k_rbgs_brick(Fine<T> F, const T *__restrict__ pin, TO *__restrict__ pout, const T *__restrict__ f,
                 const T *__restrict__ lamp, int ntx, int nty, int bx, int xoff, int ntiles) {
    constexpr int LW = 64 / RPW, NT = NW * RPW, HZO = BZ > 1 ? 2 : 0;  // lanes of a row, row takers
    constexpr int HY = BY + 4, HZ = BZ + 2 * HZO, ROWS = HY * HZ, NL = (ROWS + NT - 1) / NT;
    constexpr int RING = BZ > 1 ? (BY + 2) * (BZ + 2) - BY * BZ : 2;
    constexpr int NI = BY * BZ / NT, NH = (RING + NT - 1) / NT, NU = NI + NH;
    static_assert(NI * NT == BY * BZ, "interior rows divide among the takers");
    constexpr bool WIDEN = sizeof(TO) != sizeof(T);
    typedef T U2 __attribute__((ext_vector_type(2)));
    typedef U2 U __attribute__((aligned(sizeof(T))));  // a pair at element alignment (odd rows)
    typedef TO W2 __attribute__((ext_vector_type(2)));
    typedef W2 W __attribute__((aligned(sizeof(TO))));
    typedef uint16_t Byte2 __attribute__((aligned(1)));
    // even and odd columns apart, so that a colour's accesses are contiguous: column 2l is
    // s[0][row][l], column 2l + 1 is s[1][row][l + 1]; s[1][row][0] and s[0][row][LW] are guards
    constexpr int P = LW + 1;
    __shared__ T s[2][ROWS][P];
    __shared__ T cy[2][HY], cz[2][HZ];
    const int per = gridDim.x >> 3;  // XCD-aware order, as in the z-march
    const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (tile >= ntiles) return;
    const int nx = F.nx, ny = F.ny, nz = F.nz, tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & (LW - 1), me = wave * RPW + (RPW == 1 ? 0 : (tid & 63) / LW);
    const int x0 = tile % ntx * bx - xoff, y0 = tile / ntx % nty * BY - 2, z0 = tile / (ntx * nty) * BZ - HZO;
    const int i = x0 + 2 * l;
    const bool in0 = i >= 0 && i < nx, in1 = i >= 0 && i + 1 < nx;
    const T lam = *lamp;
    // Loads are unconditional, at places clamped into the grid: a value from outside its place
    // only meets the zero coefficients of a wall.  A pair is clamped to the row's last two cells;
    // on an odd row's last column (shf) the thread's first cell is then the second of the two.
    const uint32_t ic = (uint32_t)min(max(i, 0), nx - 2);
    const bool shf = i == nx - 1;
    auto cell = [&](int y, int z) -> uint32_t {  // fits 24 bits (by_bricks)
        const uint32_t j = (uint32_t)min(max(y0 + y, 0), ny - 1), k = (uint32_t)min(max(z0 + z, 0), nz - 1);
        return __umul24(__umul24(k, (uint32_t)ny) + j, (uint32_t)nx);
    };
    U v[NL];
    {
        int y = me % HY, z = me / HY;
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            v[q] = *reinterpret_cast<const U *>(pin + (cell(y, z) + ic));
            y += NT % HY;
            z += NT / HY;
            if (y >= HY) {
                y -= HY;
                ++z;
            }
        }
    }
    // the rows this taker updates, their right-hand sides and types
    int yu[NU], zu[NU];
    U fv[NU];
    uint32_t ty[NU];
#pragma unroll
    for (int q = 0; q < NU; ++q) {
        bool any = true;
        if (q < NI) {
            const int e = q * NT + me;
            yu[q] = e % BY + 2;
            zu[q] = e / BY + HZO;
        } else {
            const int e = (q - NI) * NT + me;  // rows beside each plane, then the rows of the end planes
            constexpr int SIDES = BZ > 1 ? 2 * (BZ + 2) : 2;
            any = e < RING;
            const int u = e - SIDES;
            yu[q] = !any ? 1 : e < SIDES ? ((e & 1) ? BY + 2 : 1) : u % BY + 2;
            zu[q] = BZ == 1 ? 0 : !any ? 1 : e < SIDES ? (e >> 1) + 1 : u / BY ? BZ + 2 : 1;
        }
        const int j = y0 + yu[q], k = z0 + zu[q];
        const bool row = any && j >= 0 && j < ny && k >= 0 && k < nz;
        const uint32_t c = cell(yu[q], zu[q]) + ic;
        fv[q] = *reinterpret_cast<const U *>(f + c);
        const uint32_t t = *reinterpret_cast<const Byte2 *>(F.type + c);
        ty[q] = (row && in0 ? (shf ? t >> 8 : t & 0xff) : T_DEAD) | (row && in1 ? t & 0xff00 : T_DEAD << 8);
        if (shf) fv[q].x = fv[q].y;
    }
    const T am[2] = {in0 ? F.axm[i] : T(0), in1 ? F.axm[i + 1] : T(0)};
    const T ap[2] = {in0 ? F.axp[i] : T(0), in1 ? F.axp[i + 1] : T(0)};
    for (int q = tid; q < HY + HZ; q += 64 * NW) {
        const int u = q < HY ? q : q - HY, g = u + (q < HY ? y0 : z0);
        const bool in = g >= 0 && g < (q < HY ? ny : nz);
        T *c = q < HY ? &cy[0][u] : &cz[0][u];
        c[0] = in ? (q < HY ? F.aym : F.azm)[g] : T(0);
        c[q < HY ? HY : HZ] = in ? (q < HY ? F.ayp : F.azp)[g] : T(0);
    }
    for (int r = tid; r < ROWS; r += 64 * NW) s[1][r][0] = s[0][r][LW] = T(0);
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int r = q * NT + me;
        if (r < ROWS) {
            s[0][r][l] = shf ? v[q].y : v[q].x;
            s[1][r][l + 1] = v[q].y;
        }
    }
    __syncthreads();
    // new value of the cell of parity b (0: first of the pair) in row (y, z), the two-pass
    // definition's operations in its order; own: the other cell of the pair
    auto update = [&](int y, int z, int b, T fc, T &own) -> T {
        const T *row = &s[0][z * HY + y][l];
        const T *c = row + (b ? ROWS * P + 1 : 0), *o = row + (b ? 0 : ROWS * P + 1);
        own = o[0];
        const T side = o[b ? 1 : -1];
        const T axm = b ? am[1] : am[0], axp = b ? ap[1] : ap[0];
        const T aym = cy[0][y], ayp = cy[1][y], azm = cz[0][z], azp = cz[1][z];
        T n = axm * (b ? own : side);
        n = n + axp * (b ? side : own);
        n = n + aym * c[-P];
        n = n + ayp * c[P];
        n = n + azm * (BZ > 1 ? c[-P * HY] : own);  // one plane: the coefficients are 0
        n = n + azp * (BZ > 1 ? c[P * HY] : own);
        T d = ((axm + axp) + aym) + ayp;
        d = d + azm;
        d = d + azp;
        return (n - (fc - lam)) / d;
    };
    // G rows at a time: their round trips overlap, and the stores keep later rows' values from
    // being fetched (and held) any earlier
    constexpr int G = 2;
    T own;
#pragma unroll
    for (int g = 0; g < NU; g += G) {
        T nv[G];
#pragma unroll
        for (int h = 0; h < G && g + h < NU; ++h) {
            const int q = g + h, b = (y0 + yu[q] + z0 + zu[q]) & 1;  // x0 is even
            nv[h] = update(yu[q], zu[q], b, b ? fv[q].y : fv[q].x, own);
        }
#pragma unroll
        for (int h = 0; h < G && g + h < NU; ++h) {
            const int q = g + h, b = (y0 + yu[q] + z0 + zu[q]) & 1;
            if ((ty[q] >> (8 * b) & 0xff) == T_FLUID) s[b][zu[q] * HY + yu[q]][l + b] = nv[h];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    const bool mine = 2 * l >= xoff && 2 * l < xoff + bx && in0;
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        const int y = yu[q], z = zu[q], b = (y0 + y + z0 + z + 1) & 1;
        const T n = update(y, z, b, b ? fv[q].y : fv[q].x, own);
        const T old = s[b][z * HY + y][l + b];
        const T x = (ty[q] >> (8 * b) & 0xff) == T_FLUID ? n : old;
        TO o0 = (TO)(b ? own : x), o1 = (TO)(b ? x : own);
        if constexpr (WIDEN) {
            if ((ty[q] & 0xff) == T_DEAD) o0 = TO(0);
            if ((ty[q] >> 8) == T_DEAD) o1 = TO(0);
        }
        const bool in = mine && y0 + y < ny && z0 + z < nz;
        TO *o = pout + cell(y, z) + i;
        if (in && in1) *reinterpret_cast<W *>(o) = W{o0, o1};
        else if (in) *o = o0;
        if ((q + 1) % G == 0) __builtin_amdgcn_sched_barrier(0);
    }
}

template <typename T, typename TO, int RPW, int BY, int BZ, int NW>
static hipError_t launch_brick(const Fine<T> &F, const T *pin, TO *pout, const T *f, const T *lam, hipStream_t s,
                               hipEvent_t ev0, hipEvent_t ev1) {
    // one tile along x needs no halo there
    constexpr int COLS = 128 / RPW;
    const int ntx = F.nx <= COLS ? 1 : (F.nx + COLS - 5) / (COLS - 4);
    const int xoff = ntx == 1 ? 0 : 2, bx = ntx == 1 ? COLS : (((F.nx + ntx - 1) / ntx + 1) & ~1);
    const int nty = (F.ny + BY - 1) / BY, ntz = (F.nz + BZ - 1) / BZ;
    const int ntiles = ntx * nty * ntz, grid = (ntiles + 7) / 8 * 8;
    if (ev0)
        hipExtLaunchKernelGGL((k_rbgs_brick<T, TO, RPW, BY, BZ, NW>), dim3(grid), dim3(64 * NW), 0, s, ev0, ev1, 0, F,
                              pin, pout, f, lam, ntx, nty, bx, xoff, ntiles);
    else
        hipLaunchKernelGGL((k_rbgs_brick<T, TO, RPW, BY, BZ, NW>), dim3(grid), dim3(64 * NW), 0, s, F, pin, pout, f,
                           lam, ntx, nty, bx, xoff, ntiles);
    return hipGetLastError();
}

// Brick shapes (FP64 us per sweep): small bricks while they give each compute unit a few (64^3: 256
// of them), 8 x 8 rows from about 10^6 cells, where the halo's work outweighs the parallelism
// (96^3 11.8 with the small ones); one row of 128 columns where it takes the place of three tiles of
// 64, 121 to 128 columns (128^3 15.9 / 18.2, 122 x 120 x 130 14.9 / 17.8, 126 x 160 x 160 26.9 / 25.9; two
// for five tiles are slower, 244 x 128 x 128 30.8 / 28.1); 16 waves of 9 rows against 8 of 18: 15.7 / 16.4.  Short rows: by their number (a V(2,2) cycle with 8 x 8 rows against 4 x 4: 13 x 160 x 160
// 213 / 230 us in FP64 but two of them 418 / 413 in FP32, 13 x 256 x 256 330 / 379 and 604 / 625).
template <typename T, typename TO>
hipError_t launch_sweep_brick(const Fine<T> &F, const T *pin, TO *pout, const T *f, const T *lam, hipStream_t s,
                              hipEvent_t ev0, hipEvent_t ev1) {
    const int64_t rows = (int64_t)F.ny * F.nz, n = F.nx * rows;
    if (F.nz == 1) return launch_brick<T, TO, 2, 8, 1, 4>(F, pin, pout, f, lam, s, ev0, ev1);
    if (n < BRICK_LARGE_CELLS && rows < BRICK_LARGE_ROWS) return launch_brick<T, TO, 2, 4, 4, 8>(F, pin, pout, f, lam, s, ev0, ev1);
    if (F.nx > 64 && F.nx <= 128 && 128 < 64 * ((F.nx + 59) / 60))
        return launch_brick<T, TO, 1, 8, 8, 16>(F, pin, pout, f, lam, s, ev0, ev1);
    return launch_brick<T, TO, 2, 8, 8, 8>(F, pin, pout, f, lam, s, ev0, ev1);
}

template hipError_t launch_sweep_brick<double, double>(const Fine<double> &, const double *, double *, const double *,
                                                       const double *, hipStream_t, hipEvent_t, hipEvent_t);
template hipError_t launch_sweep_brick<float, float>(const Fine<float> &, const float *, float *, const float *,
                                                     const float *, hipStream_t, hipEvent_t, hipEvent_t);
template hipError_t launch_sweep_brick<float, double>(const Fine<float> &, const float *, double *, const float *,
                                                      const float *, hipStream_t, hipEvent_t, hipEvent_t);

}  // namespace ibm
