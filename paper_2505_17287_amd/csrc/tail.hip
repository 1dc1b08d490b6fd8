// The tail of the V-cycle (paper Section 2.1: multigrid for the pressure equation): every level
// from the first one with at most SMALL_LEVEL cells down to the coarsest, in one workgroup.
//
// Pre-smoothing, residual and restriction, the coarsest sweeps with mean removal, prolongation
// and post-smoothing run with iterates and right-hand sides in LDS, separated by workgroup
// barriers.  One compute unit holds all of it, so the kernel is bound by that unit's
// instruction issue and by the round trips of its loads, not by bandwidth.  Hence:
// - What depends on the geometry alone is prepared per cell when the hierarchy is built
//   (k_tail_tables): the six face transmissibilities, the reciprocal diagonal, the volume, the
//   prolongation weights with the contributors' offsets and activity, the children's places.
//   A leg then starts with one round of independent loads; the index divisions, FP64 divisions
//   and table look-ups per cell and leg are gone.
// - A thread owns pairs of x neighbours, one cell of each colour, so a colour pass keeps every
//   lane busy (cells dealt out linearly left half of them masked).
// 128^3 with four bodies (levels of 10^3 and below): 47 -> 29 us; a 128^2 grid (levels 64^2 and
// below): 93 -> 58 us; 384^3: 81 -> 54 us.
// Per cell the arithmetic is that of the level-by-level sweeps (times the reciprocal of the
// diagonal), restrictions and prolongations.
#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "ibm_impl.hpp"

namespace ibm {

constexpr int TAIL_NT = 1024;

// Tables and iterates are laid out in the order the threads take the cells, so the loads of a
// wave are contiguous and its LDS accesses free of bank conflicts.  Levels of at most 64 cells
// (one wave), and those with more than 2 TAIL_NT x pairs (some odd row lengths), are in linear
// order; the others by pairs, all red cells first, then all black ones.
// n = number of cells a thread owns, negative for the linear order.
constexpr int TAIL_LIN = SMALL_LEVEL / TAIL_NT;
__host__ __device__ inline int tail_form(const int n[3]) {
    const int nc = n[0] * n[1] * n[2], pairs = ((n[0] + 1) >> 1) * n[1] * n[2];
    return nc <= 64 ? -1 : pairs <= TAIL_NT ? 2 : pairs <= 2 * TAIL_NT ? 4 : -TAIL_LIN;
}
__host__ __device__ inline int tail_span(const int n[3]) {  // table entries of a level
    return tail_form(n) < 0 ? n[0] * n[1] * n[2] : 2 * ((n[0] + 1) >> 1) * n[1] * n[2];
}

// meta.x: parent in the next coarser level (12 bits), per axis whether the second contributor of
// the prolongation is none, the one below or the one above (2 bits each), and
constexpr uint32_t TM_ALL = 1u << 18;     // every contributor is active
constexpr uint32_t TM_ACTIVE = 1u << 19;  // the cell is active
constexpr uint32_t TM_BLACK = 1u << 20;   // (I + J + K) odd
constexpr uint32_t TM_ODDX = 1u << 21;    // I odd
constexpr uint32_t TM_NONE = ~0u;         // no cell at this entry
// meta.y: the cell.  down, per cell: first child in the next finer level (12 bits), then one
// bit per axis: two children.

int tail_first(const LevelHost *lev, int nlev) {
    const int Lc = nlev - 1;
    for (int l = 1; l <= Lc; ++l) {
        if (lev[l].ncell() > SMALL_LEVEL || Lc - l + 1 > TAIL_MAX) continue;
        int64_t below = 0;
        for (int q = l + 1; q <= Lc; ++q) below += tail_span(lev[q].n);
        if (below <= TAIL_E - SMALL_LEVEL) return l;
    }
    return nlev;
}

struct TailBuild {
    int nl, total;
    int n[TAIL_MAX][3], off[TAIL_MAX], tab[TAIL_MAX];
    const uint8_t *active[TAIL_MAX];
    const double *T64[TAIL_MAX][3], *w64[TAIL_MAX][3];
    const float *T32[TAIL_MAX][3], *w32[TAIL_MAX][3];
    const int *lo[TAIL_MAX][3], *hi[TAIL_MAX][3], *cs[TAIL_MAX][3];  // cs: children in the level above
    const double *pt[TAIL_MAX][3];
    TailTables t;
};

template <typename T>
__device__ void tail_coef(const T *const *Tl, const T *const *w, const int *n, int id, const int I[3], T *coef, int at) {
    const int sy = n[0], sz = n[0] * n[1];
    const T txm = Tl[0][id], txp = I[0] < n[0] - 1 ? Tl[0][id + 1] : T(0);
    const T tym = Tl[1][id], typ = I[1] < n[1] - 1 ? Tl[1][id + sy] : T(0);
    const T tzm = Tl[2][id], tzp = I[2] < n[2] - 1 ? Tl[2][id + sz] : T(0);
    T d = txm + txp;
    d = d + tym;
    d = d + typ;
    d = d + tzm;
    d = d + tzp;
    const T c[8] = {txm, txp, tym, typ, tzm, tzp, d > T(0) ? T(1) / d : T(0), (w[0][I[0]] * w[1][I[1]]) * w[2][I[2]]};
    for (int q = 0; q < 8; ++q) coef[q * TAIL_E + at] = c[q];
}

__global__ void k_tail_tables(TailBuild B) {
    const int at = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (at >= B.total) return;
    int q = 0;
    while (q + 1 < B.nl && at >= B.tab[q + 1]) ++q;
    const int *n = B.n[q];
    int I[3], e = at - B.tab[q];
    if (tail_form(n) < 0) {
        I[0] = e % n[0];
        I[1] = e / n[0] % n[1];
        I[2] = e / (n[0] * n[1]);
    } else {
        const int hx = (n[0] + 1) >> 1, pairs = hx * n[1] * n[2], black = e >= pairs;
        e -= black ? pairs : 0;
        I[1] = e / hx % n[1];
        I[2] = e / (hx * n[1]);
        I[0] = 2 * (e % hx) + ((I[1] + I[2] + black) & 1);
    }
    if (I[0] >= n[0]) {
        B.t.meta[at] = make_uint2(TM_NONE, 0u);
        return;
    }
    const int id = (I[2] * n[1] + I[1]) * n[0] + I[0];
    tail_coef<double>(B.T64[q], B.w64[q], n, id, I, B.t.c64, at);
    tail_coef<float>(B.T32[q], B.w32[q], n, id, I, B.t.c32, at);
    uint32_t m = (((I[0] + I[1] + I[2]) & 1) ? TM_BLACK : 0) | ((I[0] & 1) ? TM_ODDX : 0);
    if (B.active[q][id]) m |= TM_ACTIVE;
    if (q + 1 < B.nl) {
        const int *c = B.n[q + 1];
        int lo[3], hi[3], step[3] = {1, c[0], c[0] * c[1]}, parent = 0;
        for (int d = 0; d < 3; ++d) {
            lo[d] = B.lo[q][d][I[d]];
            hi[d] = B.hi[q][d][I[d]];
            parent += lo[d] * step[d];
            m |= (uint32_t)(hi[d] < lo[d] ? 1 : hi[d] > lo[d] ? 2 : 0) << (12 + 2 * d);
            B.t.w[d * TAIL_E + at] = B.pt[q][d][I[d]];
        }
        bool all = true;
        for (int z = 0; z < (lo[2] == hi[2] ? 1 : 2); ++z)
            for (int y = 0; y < (lo[1] == hi[1] ? 1 : 2); ++y)
                for (int x = 0; x < (lo[0] == hi[0] ? 1 : 2); ++x)
                    if (!B.active[q + 1][(z ? hi[2] : lo[2]) * step[2] + (y ? hi[1] : lo[1]) * step[1] + (x ? hi[0] : lo[0])])
                        all = false;
        m |= (uint32_t)parent | (all ? TM_ALL : 0);
    }
    B.t.meta[at] = make_uint2(m, (uint32_t)id);
    if (q > 0) {
        const int *f = B.n[q - 1];
        const int step[3] = {1, f[0], f[0] * f[1]};
        int first = 0;
        uint32_t two = 0;
        for (int d = 0; d < 3; ++d) {
            const int a = B.cs[q][d][I[d]];
            first += a * step[d];
            if (B.cs[q][d][I[d] + 1] - a == 2) two |= 1u << (12 + d);
        }
        B.t.down[B.off[q] + id] = (uint32_t)first | two;
    }
}

hipError_t launch_tail_tables(ibm_grid *g, hipStream_t s) {
    const int lt = tail_first(g->lev, g->nlev);
    if (lt >= g->nlev) return hipSuccess;
    TailBuild B;
    B.nl = g->nlev - lt;
    B.total = 0;
    int off = 0;
    for (int q = 0; q < B.nl; ++q) {
        const LevelHost &L = g->lev[lt + q];
        B.off[q] = off;
        off += (int)L.ncell();
        B.tab[q] = B.total;
        B.total += tail_span(L.n);
        B.active[q] = L.active;
        for (int d = 0; d < 3; ++d) {
            B.n[q][d] = L.n[d];
            B.T64[q][d] = L.T64[d];
            B.T32[q][d] = L.T32[d];
            B.w64[q][d] = L.w64[d];
            B.w32[q][d] = L.w32[d];
            B.lo[q][d] = L.plo[d];
            B.hi[q][d] = L.phi[d];
            B.pt[q][d] = L.pt[d];
            B.cs[q][d] = L.cs_d[d];
        }
    }
    B.t = g->tail;
    hipLaunchKernelGGL(k_tail_tables, dim3((B.total + 127) / 128), dim3(128), 0, s, B);
    return hipGetLastError();
}

struct TailLevel {
    int n[3], off, tab;  // sizes, first cell, first table entry
};

template <typename T>
struct TailArgs {
    int nl;                                // levels; index 0 is the first, nl - 1 the coarsest
    TailLevel lev[TAIL_MAX];
    int ntab;                              // table entries of all levels
    const T *coef;                         // 8 arrays of TAIL_E: faces -x +x -y +y -z +z, 1 / diagonal, volume
    const double *w;                       // 3 arrays of TAIL_E: weight of the second contributor
    const uint2 *meta;
    const uint32_t *down;
    T *R;                                  // right-hand side of the first level
    T *e;                                  // and its correction (out)
    const double *vol;                     // summed active volume per level
    const double *partials;                // restriction partials of the first level
    int nparts, nu1, nu2, ncoarse;
};

template <typename T>
struct TailShared {
    T es[TAIL_E];                // iterates of all levels, by table entry
    T x[SMALL_LEVEL];            // by cell: the residual to restrict, or the iterate to prolong
    T R[TAIL_E - SMALL_LEVEL];   // by cell: right-hand sides of the levels below the first
    double sum[TAIL_NT / 64], mean, mu[TAIL_MAX], vol[TAIL_MAX];
    TailLevel lev[TAIL_MAX];     // a copy of the arguments' that can be indexed at run time
    __device__ __forceinline__ TailLevel level(int q) const {
        TailLevel L;
        for (int d = 0; d < 3; ++d) L.n[d] = __builtin_amdgcn_readfirstlane(lev[q].n[d]);
        L.off = __builtin_amdgcn_readfirstlane(lev[q].off);
        L.tab = __builtin_amdgcn_readfirstlane(lev[q].tab);
        return L;
    }
};

// the cells of one level that a thread owns
template <typename T, int NS>
struct TailCells {
    T t[NS][6], inv[NS], rhs[NS];
    uint32_t m[NS];
    int id[NS];
    __device__ __forceinline__ bool live(int k) const { return m[k] != TM_NONE; }
    __device__ __forceinline__ bool active(int k) const { return live(k) && (m[k] & TM_ACTIVE); }
};

// A thread's cells of a level of sizes n: entry(k) of slot k.  PAIRS: slots 2h and 2h + 1 are the
// red and the black cell of x pair tid + TAIL_NT h; else slot k is entry tid + TAIL_NT k.
template <bool PAIRS>
struct TailPlace {
    int n, hx, hz;  // pairs or cells; strides of a row and a plane of them
    __device__ __forceinline__ TailPlace(const TailLevel &L) {
        hx = PAIRS ? (L.n[0] + 1) >> 1 : L.n[0];
        hz = hx * L.n[1];
        n = hz * L.n[2];
    }
    __device__ __forceinline__ int at(int k) const { return (int)threadIdx.x + TAIL_NT * (PAIRS ? k >> 1 : k); }
    __device__ __forceinline__ bool in(int k) const { return at(k) < n; }
    __device__ __forceinline__ int pos(int k) const { return in(k) ? at(k) : 0; }
    __device__ __forceinline__ int entry(int k) const { return pos(k) + (PAIRS && (k & 1) ? n : 0); }
    // sum of T_f e_nb in the order -x +x -y +y -z +z; the transmissibility of a missing
    // neighbour is 0 and its place is clamped into the level
    template <typename T, int NS>
    __device__ __forceinline__ T sum(const TailCells<T, NS> &c, int k, const T *es) const {
        int p = pos(k);
        asm volatile("" : "+v"(p));  // keeps the six addresses from being held across the sweeps
        const int last = n - 1;
        const bool odd = PAIRS && (c.m[k] & TM_ODDX);
        const T *o = es + (PAIRS && !(k & 1) ? n : 0);  // the other colour's cells
        T s = 0;
        s = s + c.t[k][0] * o[odd ? p : max(p - 1, 0)];
        s = s + c.t[k][1] * o[PAIRS && !odd ? p : min(p + 1, last)];
        s = s + c.t[k][2] * o[max(p - hx, 0)];
        s = s + c.t[k][3] * o[min(p + hx, last)];
        s = s + c.t[k][4] * o[max(p - hz, 0)];
        s = s + c.t[k][5] * o[min(p + hz, last)];
        return s;
    }
};

// loads of a level; rhs holds the volume until tail_rhs
template <typename T, int NS, bool PAIRS>
__device__ __forceinline__ void tail_fetch(const TailArgs<T> &A, int tab, const TailPlace<PAIRS> &P,
                                           TailCells<T, NS> &c) {
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const int at = tab + P.entry(k);
        const uint2 m = A.meta[at];
#pragma unroll
        for (int f = 0; f < 6; ++f) c.t[k][f] = A.coef[f * TAIL_E + at];
        c.inv[k] = A.coef[6 * TAIL_E + at];
        c.rhs[k] = A.coef[7 * TAIL_E + at];
        c.m[k] = P.in(k) ? m.x : TM_NONE;
        c.id[k] = (int)m.y;
    }
}
template <typename T, int NS>
__device__ __forceinline__ void tail_rhs(const T *R, T mu, TailCells<T, NS> &c) {
#pragma unroll
    for (int k = 0; k < NS; ++k) c.rhs[k] = R[c.id[k]] - c.rhs[k] * mu;
}

// es += the prolonged correction ec (by cell) of the next coarser level C: trilinear from the nearest coarser
// centres, or the parent's value when one of them is inactive
template <typename T, int NS, bool PAIRS>
__device__ __forceinline__ void tail_prolong(const TailArgs<T> &A, int tab, const TailPlace<PAIRS> &P, T *es,
                                             const TailLevel &C, const T *ec, const TailCells<T, NS> &c) {
    const int cy = C.n[0], cz = C.n[0] * C.n[1];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const double *w = A.w + tab + P.entry(k);
        const double tx = w[0], ty = w[TAIL_E], tz = w[2 * TAIL_E];
        const uint32_t m = c.m[k];
        if (!c.active(k)) continue;
        const int par = (int)(m & 0xfff);
        double sv;
        if (m & TM_ALL) {
            // a missing second contributor has weight 0 and the parent's place
            const int ox = (int)((m >> 13) & 1) - (int)((m >> 12) & 1);
            const int oy = ((int)((m >> 15) & 1) - (int)((m >> 14) & 1)) * cy;
            const int oz = ((int)((m >> 17) & 1) - (int)((m >> 16) & 1)) * cz;
            const double wx[2] = {1.0 - tx, tx}, wy[2] = {1.0 - ty, ty}, wz[2] = {1.0 - tz, tz};
            sv = 0.0;
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        sv += (wx[x] * wy[y]) * wz[z] * (double)ec[par + (x ? ox : 0) + (y ? oy : 0) + (z ? oz : 0)];
        } else {
            sv = (double)ec[par];
        }
        es[P.entry(k)] = (T)((double)es[P.entry(k)] + sv);
    }
}

// ns red-black sweeps of a level; zero: es is 0 so far, so the first red pass needs no neighbours
template <typename T, int NS, bool PAIRS>
__device__ __forceinline__ void tail_sweep(const TailPlace<PAIRS> &P, T *es, int ns, bool zero, const TailCells<T, NS> &c) {
    if constexpr (NS == 1) {
        // at most 64 cells: the first wave sweeps in registers, one cell per lane, neighbours by
        // lane permutation, no LDS store or barrier per colour
        const int tid = (int)threadIdx.x;
        if (tid < 64) {
            const int lxm = max(tid - 1, 0), lxp = min(tid + 1, 63), lym = max(tid - P.hx, 0), lyp = min(tid + P.hx, 63),
                      lzm = max(tid - P.hz, 0), lzp = min(tid + P.hz, 63);
            const bool relax = c.active(0) && c.inv[0] > T(0);
            const int black = (c.m[0] & TM_BLACK) ? 1 : 0;
            T x = c.live(0) ? es[tid] : T(0);
            for (int sw = 0; sw < 2 * ns; ++sw) {
                const T xm = __shfl(x, lxm, 64), xp = __shfl(x, lxp, 64), ym = __shfl(x, lym, 64),
                        yp = __shfl(x, lyp, 64), zm = __shfl(x, lzm, 64), zp = __shfl(x, lzp, 64);
                T s = 0;
                s = s + c.t[0][0] * xm;
                s = s + c.t[0][1] * xp;
                s = s + c.t[0][2] * ym;
                s = s + c.t[0][3] * yp;
                s = s + c.t[0][4] * zm;
                s = s + c.t[0][5] * zp;
                if (relax && black == (sw & 1)) x = (s - c.rhs[0]) * c.inv[0];
            }
            if (c.live(0)) es[tid] = x;
        }
        __syncthreads();
    } else {
        for (int sw = 0; sw < ns; ++sw) {
#pragma unroll
            for (int col = 0; col < 2; ++col) {
                T v[NS];
                if (zero && sw == 0 && col == 0) {
#pragma unroll
                    for (int k = 0; k < NS; k += PAIRS ? 2 : 1) v[k] = (T(0) - c.rhs[k]) * c.inv[k];
                } else {
#pragma unroll
                    for (int k = PAIRS ? col : 0; k < NS; k += PAIRS ? 2 : 1)
                        v[k] = (P.sum(c, k, es) - c.rhs[k]) * c.inv[k];
                }
#pragma unroll
                for (int k = PAIRS ? col : 0; k < NS; k += PAIRS ? 2 : 1)
                    if (c.active(k) && c.inv[k] > T(0) && (PAIRS || ((c.m[k] & TM_BLACK) != 0) == (col != 0)))
                        es[P.entry(k)] = v[k];
                __syncthreads();
            }
        }
    }
}

// out = sum of v over the workgroup / vol (0 if that is 0); one_wave: only the first wave's
// values count
template <typename T>
__device__ __forceinline__ void tail_average(double v, bool one_wave, double vol, double *out, TailShared<T> &S) {
    const double tot = one_wave ? wave_sum(v) : block_sum<TAIL_NT>(v, S.sum, threadIdx.x);
    if (threadIdx.x == 0) *out = vol > 0.0 ? tot / vol : 0.0;
    __syncthreads();
}

// removal of the volume-weighted active mean (coarsest level); vol: the cells' volumes
template <typename T, int NS, bool PAIRS>
__device__ __forceinline__ void tail_mean(int q, const TailPlace<PAIRS> &P, T *es, TailShared<T> &S,
                                          const TailCells<T, NS> &c, const T *vol) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k)
        if (c.active(k)) acc += (double)vol[k] * (double)es[P.entry(k)];
    tail_average<T>(acc, NS == 1, S.vol[q], &S.mean, S);
    const T mean = (T)S.mean;
#pragma unroll
    for (int k = 0; k < NS; ++k)
        if (c.active(k)) es[P.entry(k)] -= mean;
}

// residual (R - V mu) - (A e) of the active cells into x, 0 elsewhere
template <typename T, int NS, bool PAIRS>
__device__ __forceinline__ void tail_residual(const TailPlace<PAIRS> &P, const T *es, T *x,
                                              const TailCells<T, NS> &c) {
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        if (!c.live(k)) continue;
        T d = c.t[k][0] + c.t[k][1];
        d = d + c.t[k][2];
        d = d + c.t[k][3];
        d = d + c.t[k][4];
        d = d + c.t[k][5];
        const T r = c.rhs[k] - (P.sum(c, k, es) - d * es[P.entry(k)]);
        x[c.id[k]] = (c.m[k] & TM_ACTIVE) ? r : T(0);
    }
}

// the thread's own iterates by cell, for the prolongation into the finer level
template <typename T, int NS, bool PAIRS>
__device__ __forceinline__ void tail_publish(const TailPlace<PAIRS> &P, const T *es, T *x, const TailCells<T, NS> &c) {
#pragma unroll
    for (int k = 0; k < NS; ++k)
        if (c.live(k)) x[c.id[k]] = es[P.entry(k)];
}

// right-hand side and mu of level q (sizes C) from the residual of the level above it (sizes F):
// children summed x fastest, then y, then z.  d0: the thread's first word of A.down, loaded ahead.
template <typename T>
__device__ __forceinline__ void tail_restrict(const TailArgs<T> &A, int q, const TailLevel &F, const TailLevel &C,
                                              T *R, TailShared<T> &S, uint32_t d0) {
    const int tid = (int)threadIdx.x, ncc = C.n[0] * C.n[1] * C.n[2];
    const int sy = F.n[0], sz = F.n[0] * F.n[1];
    double psum = 0.0;
    for (int id = tid; id < ncc; id += TAIL_NT) {
        const uint32_t d = id == tid ? d0 : A.down[C.off + id];
        const int a = (int)(d & 0xfff);
        T r = 0;
        for (int k = 0; k <= (int)((d >> 14) & 1); ++k)
            for (int j = 0; j <= (int)((d >> 13) & 1); ++j)
                for (int i = 0; i <= (int)((d >> 12) & 1); ++i) r += S.x[a + k * sz + j * sy + i];
        R[id] = r;
        psum += (double)r;
    }
    tail_average<T>(psum, ncc <= 64, S.vol[q], &S.mu[q], S);
}

// One leg of level q.  On the way down its right-hand side is formed while its tables are in
// flight; on return S.x holds its residual (down) or its iterate (coarsest level, and up).
template <typename T, int NS, bool PAIRS>
__device__ __forceinline__ void tail_leg(const TailArgs<T> &A, int q, const TailLevel &L, TailShared<T> &S, bool up) {
    const int tid = (int)threadIdx.x;
    T *es = S.es + L.tab;
    const TailPlace<PAIRS> P(L);
    const bool coarsest = q + 1 == A.nl;
    const TailLevel N = S.level(up ? q + 1 : max(q - 1, 0));  // the level the leg takes from
    TailCells<T, NS> c;
    tail_fetch<T, NS, PAIRS>(A, L.tab, P, c);
    T *R = q == 0 ? A.R : S.R + (L.off - S.level(1).off);
    if (!up) {
        if (q == 0) {  // mu from the fine restriction's partials
            double a = 0.0;
            for (int k = tid; k < A.nparts; k += TAIL_NT) a += A.partials[k];
            tail_average<T>(a, false, S.vol[0], &S.mu[0], S);
        } else {
            tail_restrict<T>(A, q, N, L, R, S, tid < L.n[0] * L.n[1] * L.n[2] ? A.down[L.off + tid] : 0);
        }
    }
    T vol[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) vol[k] = c.rhs[k];
    tail_rhs<T, NS>(R, (T)S.mu[q], c);
    if (up) {
        tail_prolong<T, NS, PAIRS>(A, L.tab, P, es, N, S.x, c);
        __syncthreads();
    }
    tail_sweep<T, NS, PAIRS>(P, es, coarsest ? A.ncoarse : up ? A.nu2 : A.nu1, !up, c);
    if (coarsest) tail_mean<T, NS, PAIRS>(q, P, es, S, c, vol);
    if (up || coarsest) tail_publish<T, NS, PAIRS>(P, es, S.x, c);
    else tail_residual<T, NS, PAIRS>(P, es, S.x, c);
    __syncthreads();
}

template <typename T>
__global__ void __launch_bounds__(TAIL_NT) k_tailC(TailArgs<T> A) {
    __shared__ TailShared<T> S;
    const int tid = (int)threadIdx.x, nl = A.nl;
#pragma unroll
    for (int q = 0; q < TAIL_MAX; ++q)
        if (tid == q) S.lev[q] = A.lev[q];
    if (tid < nl) S.vol[tid] = A.vol[tid];
    for (int at = tid; at < A.ntab; at += TAIL_NT) S.es[at] = T(0);
    // one word of every 128-byte line of the deeper levels' tables, so that their legs find them
    // in L2 (the fine level's passes have streamed it out since the last cycle)
    constexpr int LINE = 128 / sizeof(T);
    for (int at = A.lev[1].tab + LINE * (tid >> 3); at < A.ntab; at += LINE * (TAIL_NT >> 3)) {
        const T warm = A.coef[(tid & 7) * TAIL_E + at];
        asm volatile("" ::"v"(warm));
    }
    __syncthreads();
    // one loop over the legs, down then up, so that each form of a leg is compiled once
    for (int leg = 0; leg < 2 * nl - 1; ++leg) {
        const int q = leg < nl ? leg : 2 * nl - 2 - leg;
        const TailLevel L = S.level(q);
        const int form = tail_form(L.n);
        if (form == -1) tail_leg<T, 1, false>(A, q, L, S, leg >= nl);
        else if (form == 2) tail_leg<T, 2, true>(A, q, L, S, leg >= nl);
        else if (form == 4) tail_leg<T, 4, true>(A, q, L, S, leg >= nl);
        else tail_leg<T, TAIL_LIN, false>(A, q, L, S, leg >= nl);
    }
    // the first level's correction goes back to global memory for the prolongation above
    const TailLevel L = S.level(0);
    for (int id = tid; id < L.n[0] * L.n[1] * L.n[2]; id += TAIL_NT) A.e[id] = S.x[id];
}

template <typename T>
hipError_t launch_tail(ibm_grid *g, int lt, const Coarse<T> &first, int nparts, const ibm_solve_opts *o,
                       hipStream_t s) {
    TailArgs<T> A;
    A.nl = g->nlev - lt;
    A.ntab = 0;
    int off = 0;
    for (int q = 0; q < A.nl; ++q) {
        for (int d = 0; d < 3; ++d) A.lev[q].n[d] = g->lev[lt + q].n[d];
        A.lev[q].off = off;
        A.lev[q].tab = A.ntab;
        off += (int)g->lev[lt + q].ncell();
        A.ntab += tail_span(A.lev[q].n);
    }
    for (int q = A.nl; q < TAIL_MAX; ++q) A.lev[q] = TailLevel{{1, 1, 1}, off, A.ntab};
    if constexpr (sizeof(T) == 8) A.coef = g->tail.c64;
    else A.coef = g->tail.c32;
    A.w = g->tail.w;
    A.meta = g->tail.meta;
    A.down = g->tail.down;
    A.R = first.R;
    A.e = first.e;
    A.vol = &g->sc->vol[lt];
    A.partials = g->partials;
    A.nparts = nparts;
    A.nu1 = o->nu1;
    A.nu2 = o->nu2;
    A.ncoarse = o->coarsest_sweeps;
    hipLaunchKernelGGL(k_tailC<T>, dim3(1), dim3(TAIL_NT), 0, s, A);
    return hipGetLastError();
}

template hipError_t launch_tail<double>(ibm_grid *, int, const Coarse<double> &, int, const ibm_solve_opts *, hipStream_t);
template hipError_t launch_tail<float>(ibm_grid *, int, const Coarse<float> &, int, const ibm_solve_opts *, hipStream_t);

}  // namespace ibm
