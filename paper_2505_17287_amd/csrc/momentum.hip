// Advection-diffusion half-step of the fractional-step method (Section 2.1): conservative
// central-difference convection (Adams-Bashforth), Crank-Nicolson viscous term solved by
// scheduled relaxed Jacobi, with the no-slip (Dirichlet) ghost rows of Section 2.2.
//
// Cell-centred velocity components live in three arrays of the level-0 layout [nz][ny][nx].
// The two cell passes (right-hand side, relaxed Jacobi sweep) march in z over tiles of columns
// (mom_march below).
#include <algorithm>
#include <type_traits>

#include "device_util.hpp"
#include "ibm_impl.hpp"

namespace ibm {

namespace {

constexpr int DREF_NT = 256;     // ghost refresh: eight lanes per ghost

struct CV3 {
    const double *c[3];
};
struct V3 {
    double *c[3];
};

struct MomView {
    int nx, ny, nz;
    const double *xc, *yc, *zc;  // centres
    const double *xf, *yf, *zf;  // faces
    const double *wx, *wy, *wz;  // widths
    const double *axm, *axp, *aym, *ayp, *azm, *azp;  // flux coefficients per unit volume
    const uint8_t *type;
};

MomView mom_view(ibm_grid *g) {
    MomView M;
    M.nx = g->nx;
    M.ny = g->ny;
    M.nz = g->nz;
    M.xc = g->c0[0];
    M.yc = g->c0[1];
    M.zc = g->c0[2];
    M.xf = g->faces[0];
    M.yf = g->faces[1];
    M.zf = g->faces[2];
    M.wx = g->w0[0];
    M.wy = g->w0[1];
    M.wz = g->w0[2];
    M.axm = g->am0[0];
    M.axp = g->ap0[0];
    M.aym = g->am0[1];
    M.ayp = g->ap0[1];
    M.azm = g->am0[2];
    M.azp = g->ap0[2];
    M.type = g->type;
    return M;
}

// Dirichlet ghost rows, one pass: u_g = (2 - betaD_g) u_BI - sum_{m != g} betaD_m u_m with
// fluid members read from dst (already updated) and ghost members from src (the values
// before the pass).  Lane m of a group of eight takes member m; three shuffle steps sum the
// group.  A degenerate ghost takes 2 u_BI minus the mean of its fluid 26-neighbours.
__global__ void __launch_bounds__(DREF_NT)
    k_dirichlet_refresh(GhostView G, const double *__restrict__ betaDg, const double *__restrict__ ubi, CV3 src,
                        V3 dst, int nx, int ny, int nz, const uint8_t *__restrict__ type, double *scr) {
    const int64_t g = ((int64_t)blockIdx.x * DREF_NT + threadIdx.x) >> 3;
    const int m = threadIdx.x & 7;
    const bool live = g < G.ng;
    const int64_t gc = live ? g : 0;
    const int32_t q = G.st[8 * gc + m];
    const double b = G.beta[8 * gc + m];  // the Dirichlet weights (ghosts() below)
    const unsigned gm = G.gmask[gc];
    double t[3] = {0.0, 0.0, 0.0};
    if (live && q >= 0) {
        const bool from_src = ((gm >> m) & 1u) != 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c] = b * (from_src ? src.c[c][q] : dst.c[c][q]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        t[c] += __shfl_xor(t[c], 1, 64);
        t[c] += __shfl_xor(t[c], 2, 64);
        t[c] += __shfl_xor(t[c], 4, 64);
    }
    if (!live || m != 0) return;
    const int64_t cell = G.cell[gc];
    const double ub[3] = {ubi[3 * gc], ubi[3 * gc + 1], ubi[3 * gc + 2]};
    if (G.flags[gc] & GF_DEGENERATE) {
        int i, j, k;
        unflatten(cell, nx, ny, i, j, k);
        double sm[3] = {0.0, 0.0, 0.0};
        int n = 0;
        for (int dk = -1; dk <= 1; ++dk)
            for (int dj = -1; dj <= 1; ++dj)
                for (int di = -1; di <= 1; ++di) {
                    const int ii = i + di, jj = j + dj, kk = k + dk;
                    if (ii < 0 || jj < 0 || kk < 0 || ii >= nx || jj >= ny || kk >= nz) continue;
                    const int64_t qq = ((int64_t)kk * ny + jj) * nx + ii;
                    if (type[qq] == T_FLUID) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) sm[c] += dst.c[c][qq];
                        ++n;
                    }
                }
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c] = 2.0 * ub[c] - (n ? sm[c] / n : 0.0);
    } else {
        const double w = 2.0 - betaDg[gc];
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c] = w * ub[c] - t[c];
    }
    if (scr) {  // values held back, scattered by k_ghost_scatter (an in-place pass)
#pragma unroll
        for (int c = 0; c < 3; ++c) scr[3 * gc + c] = t[c];
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) dst.c[c][cell] = t[c];
    }
}

__global__ void k_ghost_scatter(int64_t ng, const int32_t *__restrict__ gcell, const double *__restrict__ scr, V3 dst) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= ng) return;
    const int64_t cell = gcell[g];
#pragma unroll
    for (int c = 0; c < 3; ++c) dst.c[c][cell] = scr[3 * g + c];
}

// March of the two cell passes.  A workgroup of NW waves owns a tile of columns and a chunk of
// planes; RPW rows of 64 / RPW lanes per wave, two adjacent columns per lane (16-byte accesses),
// the first and the last row of the tile being halo rows that only supply values.  A thread keeps
// the pairs of three planes of the three components in registers and loads one plane ahead; the
// current plane goes through LDS for the x and y neighbours (even and odd columns apart, so that
// a wave's reads are contiguous; one barrier a plane, double-buffered), so nothing is loaded
// twice but the halo.  Both passes are bound by HBM (73 and 97 bytes per cell).  With one column per
// thread and every neighbour loaded (26 and 39 loads a plane, 150 and 208 registers) they took 314 and
// 540 us at 256^3; this way 267 and 408 us.
struct MTiles {
    int ntx, nty, bx, kc, ntiles, grid;
};

template <int RPW, int NW>
struct March {
    static constexpr int LW = 64 / RPW, ROWS = NW * RPW, BY = ROWS - 2, P = LW + 1;
    typedef double U2 __attribute__((ext_vector_type(2)));
    typedef U2 U __attribute__((aligned(8)));  // a pair at element alignment (odd rows)
    typedef uint16_t Byte2 __attribute__((aligned(1)));
    struct Shared {
        double s[2][3][2][ROWS][P];  // buffer, component, even / odd columns (guards: odd 0, even LW)
    };
    int nx, ny, nz, l, r, i, j, k0, k1;
    bool live, in0, in1, mine, shf, edge;
    uint32_t ic, xe;      // first column of the loaded pair; the column beside the tile (edge lanes)
    int64_t plane, row;

    __device__ __forceinline__ March(const MTiles &t, int nx_, int ny_, int nz_) : nx(nx_), ny(ny_), nz(nz_) {
        const int per = gridDim.x >> 3;  // XCD-aware order (see zmarch.hpp)
        const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
        live = tile < t.ntiles;
        const int wave = (int)threadIdx.x >> 6;
        l = (int)threadIdx.x & (LW - 1);
        r = wave * RPW + (RPW == 1 ? 0 : ((int)threadIdx.x & 63) / LW);
        i = tile % t.ntx * t.bx + 2 * l;
        j = tile / t.ntx % t.nty * BY + r - 1;
        k0 = tile / (t.ntx * t.nty) * t.kc;
        k1 = min(nz, k0 + t.kc);
        const bool rowin = j >= 0 && j < ny && r >= 1 && r <= BY && 2 * l < t.bx;
        in0 = rowin && i < nx;
        in1 = rowin && i + 1 < nx;
        mine = in0;
        shf = i == nx - 1;
        ic = (uint32_t)min(i, nx - 2);
        edge = l == 0 || l == LW - 1;
        xe = (uint32_t)(l == 0 ? max(i - 1, 0) : min(i + 2, nx - 1));
        plane = (int64_t)nx * ny;
        row = (int64_t)min(max(j, 0), ny - 1) * nx;
    }
    __device__ __forceinline__ int64_t base(int k) const { return (int64_t)min(max(k, 0), nz - 1) * plane + row; }
    __device__ __forceinline__ U pair(const double *a, int64_t b) const {
        return *reinterpret_cast<const U *>(a + b + ic);
    }
    __device__ __forceinline__ U fix(U v) const {  // an odd row's last column is the second of the loaded pair
        if (shf) v.x = v.y;
        return v;
    }
    __device__ __forceinline__ void store(double *a, int64_t b, double v0, double v1) const {
        typedef double W2 __attribute__((ext_vector_type(2)));
        typedef W2 W __attribute__((aligned(8)));
        if (in1) __builtin_nontemporal_store(W{v0, v1}, reinterpret_cast<W *>(a + b + i));
        else __builtin_nontemporal_store(v0, a + b + i);
    }
};

// Runs body(k, below, centre, above, f, type, nb) over the chunk; nb(c, b, q): component c of the
// neighbour of cell b (0, 1) at -x, +x, -y, +y (q).  F: a second field, read at the cell itself
// (not loaded when its components are null).
template <int RPW, int NW, typename Body>
__device__ __forceinline__ void mom_march(const March<RPW, NW> &m, typename March<RPW, NW>::Shared &sh, CV3 X, CV3 F,
                                          const uint8_t *type, Body body) {
    using U = typename March<RPW, NW>::U;
    constexpr int LW = March<RPW, NW>::LW;
    struct Own {  // what only its own step needs, loaded one plane ahead
        U f[3];
        double e[3];
        uint32_t t;
    };
    auto own = [&](int k) {
        Own d;
        const int64_t b = m.base(k);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            d.f[c] = U{0.0, 0.0};
            if (F.c[0] && m.mine) d.f[c] = m.pair(F.c[c], b);
            d.e[c] = m.edge ? X.c[c][b + m.xe] : 0.0;
        }
        d.t = *reinterpret_cast<const typename March<RPW, NW>::Byte2 *>(type + b + m.ic);
        return d;
    };
    U below[3], centre[3], next[3];
    {
        const int64_t b0 = m.base(m.k0 - 1), b1 = m.base(m.k0), b2 = m.base(m.k0 + 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            below[c] = m.fix(m.pair(X.c[c], b0));
            centre[c] = m.fix(m.pair(X.c[c], b1));
            next[c] = m.pair(X.c[c], b2);
        }
    }
    Own o = own(m.k0);
    int buf = 0;
    for (int k = m.k0; k < m.k1; ++k, buf ^= 1) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            sh.s[buf][c][0][m.r][m.l] = centre[c].x;
            sh.s[buf][c][1][m.r][m.l + 1] = centre[c].y;
            if (m.l == 0) sh.s[buf][c][1][m.r][0] = o.e[c];
            if (m.l == LW - 1) sh.s[buf][c][0][m.r][LW] = o.e[c];
        }
        U ahead[3];
        const int64_t b2 = m.base(k + 2);
#pragma unroll
        for (int c = 0; c < 3; ++c) ahead[c] = m.pair(X.c[c], b2);
        const Own on = own(k + 1);
        __syncthreads();
        U above[3], f[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            above[c] = m.fix(next[c]);
            f[c] = m.fix(o.f[c]);
        }
        if (m.mine) {
            auto nb = [&](int c, int b, int q) -> double {
                const double(&s)[2][March<RPW, NW>::ROWS][March<RPW, NW>::P] = sh.s[buf][c];
                if (q == 0) return b ? centre[c].x : s[1][m.r][m.l];
                if (q == 1) return b ? s[0][m.r][m.l + 1] : centre[c].y;
                return s[b][m.r + (q == 2 ? -1 : 1)][m.l + b];
            };
            body(k, below, centre, above, f, m.shf ? o.t >> 8 : o.t, nb);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            below[c] = centre[c];
            centre[c] = above[c];
            next[c] = ahead[c];
        }
        o = on;
    }
}

// Right-hand side of the Crank-Nicolson system on fluid rows and the convective term:
//   H = -(1/V) sum_faces (+/-) A_f Un_f (u_i)_f      (face values: linear interpolation)
//   b = u + dt (3/2 H - 1/2 H_old) + a L u,   a = nu dt / 2   (first step: H_old = H)
// H overwrites H_old in place (each thread reads and writes only its own cells; a plane of H_old
// is read before the plane of H below it is written, and no cell is read twice).  Non-fluid
// cells get H = b = 0.  partials[block] = sum of b^2 over the block's fluid cells.
constexpr int MOM_KC_MAX = 256;
template <int RPW, int NW>
__global__ void __launch_bounds__(64 * NW)
    k_mom_rhs(MomView M, CV3 U, V3 H, V3 B, double dt, double a, int first, MTiles t, double *partials) {
    __shared__ typename March<RPW, NW>::Shared sh;
    __shared__ double red[NW], zw[7][MOM_KC_MAX];  // per plane: four face weights, width, two coefficients
    __shared__ double xw[7][2][March<RPW, NW>::LW];  // the same per column, even and odd ones
    const March<RPW, NW> m(t, M.nx, M.ny, M.nz);
    if (!m.live) {
        if (threadIdx.x == 0) partials[blockIdx.x] = 0.0;
        return;
    }
    for (int q = (int)threadIdx.x; q < m.k1 - m.k0; q += 64 * NW) {
        const int k = m.k0 + q;
        double w[4] = {0.0, 0.0, 0.0, 0.0};
        if (k < m.nz - 1) {
            const double h = M.zc[k + 1] - M.zc[k];
            w[0] = (M.zc[k + 1] - M.zf[k + 1]) / h;
            w[1] = (M.zf[k + 1] - M.zc[k]) / h;
        }
        if (k > 0) {
            const double h = M.zc[k] - M.zc[k - 1];
            w[2] = (M.zc[k] - M.zf[k]) / h;
            w[3] = (M.zf[k] - M.zc[k - 1]) / h;
        }
        for (int v = 0; v < 4; ++v) zw[v][q] = w[v];
        zw[4][q] = M.wz[k];
        zw[5][q] = k > 0 ? M.azm[k] : 0.0;
        zw[6][q] = k < m.nz - 1 ? M.azp[k] : 0.0;
    }
    // interpolation weights (low cell, high cell) and flux coefficients; 0 on the walls
    if (m.r == 0) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int i = min(m.i + b, m.nx - 1);
            double w[4] = {0.0, 0.0, 0.0, 0.0};
            if (i < m.nx - 1) {
                const double h = M.xc[i + 1] - M.xc[i];
                w[0] = (M.xc[i + 1] - M.xf[i + 1]) / h;
                w[1] = (M.xf[i + 1] - M.xc[i]) / h;
            }
            if (i > 0) {
                const double h = M.xc[i] - M.xc[i - 1];
                w[2] = (M.xc[i] - M.xf[i]) / h;
                w[3] = (M.xf[i] - M.xc[i - 1]) / h;
            }
            for (int v = 0; v < 4; ++v) xw[v][b][m.l] = w[v];
            xw[4][b][m.l] = M.wx[i];
            xw[5][b][m.l] = i > 0 ? M.axm[i] : 0.0;
            xw[6][b][m.l] = i < m.nx - 1 ? M.axp[i] : 0.0;
        }
    }
    const int j = min(max(m.j, 0), m.ny - 1);
    double ypl = 0, yph = 0, yml = 0, ymh = 0, cym = 0, cyp = 0;
    if (j < m.ny - 1) {
        const double h = M.yc[j + 1] - M.yc[j];
        ypl = (M.yc[j + 1] - M.yf[j + 1]) / h;
        yph = (M.yf[j + 1] - M.yc[j]) / h;
        cyp = M.ayp[j];
    }
    if (j > 0) {
        const double h = M.yc[j] - M.yc[j - 1];
        yml = (M.yc[j] - M.yf[j]) / h;
        ymh = (M.yf[j] - M.yc[j - 1]) / h;
        cym = M.aym[j];
    }
    const double wy = M.wy[j];
    CV3 hold;
    for (int c = 0; c < 3; ++c) hold.c[c] = first ? nullptr : H.c[c];
    __syncthreads();
    double acc = 0.0;
    using P = typename March<RPW, NW>::U;
    mom_march<RPW, NW>(m, sh, U, hold, M.type,
                       [&](int k, const P(&below)[3], const P(&centre)[3], const P(&above)[3], const P(&hf)[3],
                           uint32_t ty, auto nb) {
        const int q = k - m.k0;
        const double zpl = zw[0][q], zph = zw[1][q], zml = zw[2][q], zmh = zw[3][q], wz = zw[4][q], czm = zw[5][q],
                     czp = zw[6][q];
        double hv[3][2], bv[3][2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const bool fluid = ((ty >> (8 * b)) & 0xff) == T_FLUID && (b ? m.in1 : true);
            const double xpl = xw[0][b][m.l], xph = xw[1][b][m.l], xml = xw[2][b][m.l], xmh = xw[3][b][m.l],
                         wx = xw[4][b][m.l], cxm = xw[5][b][m.l], cxp = xw[6][b][m.l];
            const double ax = wz * wy, ay = wz * wx, az = wy * wx, vol = (wz * wy) * wx;
            auto at = [&](const P(&v)[3], int c) { return b ? v[c].y : v[c].x; };
            const double uxp = xpl * at(centre, 0) + xph * nb(0, b, 1);
            const double uxm = xml * nb(0, b, 0) + xmh * at(centre, 0);
            const double vyp = ypl * at(centre, 1) + yph * nb(1, b, 3);
            const double vym = yml * nb(1, b, 2) + ymh * at(centre, 1);
            const double wzp = zpl * at(centre, 2) + zph * at(above, 2);
            const double wzm = zml * at(below, 2) + zmh * at(centre, 2);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double fc = at(centre, c), fxm = nb(c, b, 0), fxp = nb(c, b, 1), fym = nb(c, b, 2),
                             fyp = nb(c, b, 3), fzm = at(below, c), fzp = at(above, c);
                // a wall's weights and coefficients are 0: its terms vanish
                double h = 0.0;
                h -= (uxp * (xpl * fc + xph * fxp)) * ax;
                h += (uxm * (xml * fxm + xmh * fc)) * ax;
                h -= (vyp * (ypl * fc + yph * fyp)) * ay;
                h += (vym * (yml * fym + ymh * fc)) * ay;
                h -= (wzp * (zpl * fc + zph * fzp)) * az;
                h += (wzm * (zml * fzm + zmh * fc)) * az;
                h /= vol;
                double lap = 0.0;
                lap += cxp * (fxp - fc);
                lap -= cxm * (fc - fxm);
                lap += cyp * (fyp - fc);
                lap -= cym * (fc - fym);
                lap += czp * (fzp - fc);
                lap -= czm * (fc - fzm);
                const double hp = first ? h : at(hf, c);
                const double rhs = fc + dt * (1.5 * h - 0.5 * hp) + a * lap;
                hv[c][b] = fluid ? h : 0.0;
                bv[c][b] = fluid ? rhs : 0.0;
                acc += bv[c][b] * bv[c][b];
            }
            __builtin_amdgcn_sched_barrier(0);  // one cell's values at a time in registers
        }
        const int64_t o = m.base(k);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            m.store(H.c[c], o, hv[c][0], hv[c][1]);
            m.store(B.c[c], o, bv[c][0], bv[c][1]);
        }
    });
    const double tot = block_sum<64 * NW>(acc, red, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// One relaxed Jacobi sweep of the fluid rows of (I - a L) u = b:
//   y = (1 - omega) x + omega (b + a sum_f a_f x_nb) / (1 + a sum_f a_f)
// ghost cells are copied (their rows follow in their own pass), dead cells cleared.
// partials[block] = sum of the squared fluid-row residuals b - (I - a L) x at the input.
template <int RPW, int NW>
__global__ void __launch_bounds__(64 * NW, 3)
    k_srj_sweep(MomView M, CV3 X, V3 Y, CV3 B, double a, double omega, MTiles t, double *partials) {
    __shared__ typename March<RPW, NW>::Shared sh;
    __shared__ double red[NW], zw[2][MOM_KC_MAX];
    const March<RPW, NW> m(t, M.nx, M.ny, M.nz);
    if (!m.live) {
        if (threadIdx.x == 0) partials[blockIdx.x] = 0.0;
        return;
    }
    for (int q = (int)threadIdx.x; q < m.k1 - m.k0; q += 64 * NW) {
        const int k = m.k0 + q;
        zw[0][q] = k > 0 ? M.azm[k] : 0.0;
        zw[1][q] = k < m.nz - 1 ? M.azp[k] : 0.0;
    }
    double cxm[2], cxp[2];  // 0 on the walls
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int i = min(m.i + b, m.nx - 1);
        cxm[b] = i > 0 ? M.axm[i] : 0.0;
        cxp[b] = i < m.nx - 1 ? M.axp[i] : 0.0;
    }
    const int j = min(max(m.j, 0), m.ny - 1);
    const double cym = j > 0 ? M.aym[j] : 0.0, cyp = j < m.ny - 1 ? M.ayp[j] : 0.0;
    __syncthreads();
    double acc = 0.0;
    using P = typename March<RPW, NW>::U;
    mom_march<RPW, NW>(m, sh, X, B, M.type,
                       [&](int k, const P(&below)[3], const P(&centre)[3], const P(&above)[3], const P(&rhs)[3],
                           uint32_t ty, auto nb) {
        const double czm = zw[0][k - m.k0], czp = zw[1][k - m.k0];
        const int64_t o = m.base(k);
        const uint32_t tc[2] = {ty & 0xff, (ty >> 8) & 0xff};
        const bool fluid[2] = {tc[0] == T_FLUID, tc[1] == T_FLUID && m.in1};
        double den[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const double d = ((czm + czp) + (cym + cyp)) + (cxm[b] + cxp[b]);
            den[b] = 1.0 + a * d;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double y[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                auto at = [&](const P(&v)[3]) { return b ? v[c].y : v[c].x; };
                double s = 0.0;
                s += cxp[b] * nb(c, b, 1);
                s += cxm[b] * nb(c, b, 0);
                s += cyp * nb(c, b, 3);
                s += cym * nb(c, b, 2);
                s += czp * at(above);
                s += czm * at(below);
                const double xc = at(centre), num = at(rhs) + a * s, r = num - den[b] * xc;
                y[b] = fluid[b] ? (1.0 - omega) * xc + omega * (num / den[b]) : tc[b] == T_DEAD ? 0.0 : xc;
                acc += fluid[b] ? r * r : 0.0;
            }
            m.store(Y.c[c], o, y[0], y[1]);
            __builtin_amdgcn_sched_barrier(0);  // one component's values at a time in registers
        }
    });
    const double tot = block_sum<64 * NW>(acc, red, threadIdx.x);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// Workgroups: the sweep four waves with three workgroups per compute unit (156 registers; eight
// waves at 128 registers spill: 460 us at 256^3), the right-hand side eight waves, one workgroup
// (251 registers; two of four waves 455, any bound on the registers 1800 us and more).
// Tiles of cols columns and by rows, `per_cu` workgroups per compute unit at once; a chunk of kc
// planes costs about kc + 3 plane steps, and the chunk count minimises rounds x (kc + 3).
MTiles mom_tiles(int nx, int ny, int nz, int cols, int by, int per_cu) {
    MTiles t;
    t.ntx = (nx + cols - 1) / cols;
    t.bx = ((nx + t.ntx - 1) / t.ntx + 1) & ~1;
    t.nty = (ny + by - 1) / by;
    const int64_t per_slab = (int64_t)t.ntx * t.nty, slots = (int64_t)per_cu * device_cu_count();
    int64_t best = -1;
    t.kc = std::min(nz, MOM_KC_MAX);
    for (int c = 1; c <= nz; ++c) {
        const int kc = (nz + c - 1) / c;
        if (kc > MOM_KC_MAX) continue;
        const int64_t cost = (per_slab * c + slots - 1) / slots * (kc + 3);
        if (best < 0 || cost < best) {
            best = cost;
            t.kc = kc;
        }
    }
    t.ntiles = (int)(per_slab * ((nz + t.kc - 1) / t.kc));
    t.grid = (t.ntiles + 7) / 8 * 8;
    return t;
}

// rows of 128 columns, or of 64 where those waste fewer lanes
bool mom_wide(int nx) { return (nx + 127) / 128 * 128 <= (nx + 63) / 64 * 64; }

__global__ void k_mom_sum(const double *partials, int n, double *out) {
    __shared__ double sh[4];
    double a = 0.0;
    for (int q = threadIdx.x; q < n; q += 256) a += partials[q];
    a = block_sum<256>(a, sh, threadIdx.x);
    if (threadIdx.x == 0) *out = a;
}

CV3 cv3(const double *a, const double *b, const double *c) {
    CV3 v;
    v.c[0] = a;
    v.c[1] = b;
    v.c[2] = c;
    return v;
}
V3 v3(double *a, double *b, double *c) {
    V3 v;
    v.c[0] = a;
    v.c[1] = b;
    v.c[2] = c;
    return v;
}

// the ghost list with the Dirichlet weights in place of the Neumann ones
GhostView ghosts(ibm_grid *g) {
    GhostView G;
    G.ng = g->ng;
    G.cell = g->g_cell;
    G.st = g->g_st;
    G.gmask = g->g_mask;
    G.beta = g->g_betaD;
    G.h = nullptr;
    G.flags = g->g_flags;
    return G;
}

hipError_t refresh(ibm_grid *g, CV3 src, V3 dst, hipStream_t s, double *scr = nullptr) {
    if (g->ng == 0) return hipSuccess;
    hipLaunchKernelGGL(k_dirichlet_refresh, dim3((unsigned)((8 * g->ng + DREF_NT - 1) / DREF_NT)), dim3(DREF_NT), 0,
                       s, ghosts(g), g->g_betaDg, g->g_ubi, src, dst, g->nx, g->ny, g->nz, g->type, scr);
    if (scr)
        hipLaunchKernelGGL(k_ghost_scatter, dim3((unsigned)((g->ng + 255) / 256)), dim3(256), 0, s, g->ng, g->g_cell,
                           scr, dst);
    return hipGetLastError();
}

// Fresh-cell values (one pass over the fresh list, members read from the field as it is):
//   u_c = (u_BI + sum_{m != c} beta_m u_m) / (2 - beta_c);
// a degenerate fresh cell takes the mean of its fluid, non-fresh 26-neighbours (u_BI if it
// has none).  Results go to scr (three per fresh cell) and are scattered afterwards.
__global__ void k_fresh_fill(int64_t nf, const int32_t *__restrict__ fcell, const int32_t *__restrict__ fst,
                             const double *__restrict__ fbeta, const double *__restrict__ fbetac,
                             const int32_t *__restrict__ fflags, const double *__restrict__ ubi, CV3 U,
                             const uint8_t *__restrict__ type, const uint8_t *__restrict__ prev, int nx, int ny,
                             int nz, double *scr) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nf) return;
    double v[3];
    if (fflags[q] & GF_DEGENERATE) {
        int i, j, k;
        unflatten(fcell[q], nx, ny, i, j, k);
        double sm[3] = {0.0, 0.0, 0.0};
        int n = 0;
        for (int dk = -1; dk <= 1; ++dk)
            for (int dj = -1; dj <= 1; ++dj)
                for (int di = -1; di <= 1; ++di) {
                    const int ii = i + di, jj = j + dj, kk = k + dk;
                    if (ii < 0 || jj < 0 || kk < 0 || ii >= nx || jj >= ny || kk >= nz) continue;
                    const int64_t x = ((int64_t)kk * ny + jj) * nx + ii;
                    if (type[x] == T_FLUID && prev[x] == T_FLUID) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) sm[c] += U.c[c][x];
                        ++n;
                    }
                }
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = n ? sm[c] / n : ubi[3 * q + c];
    } else {
        double acc[3] = {0.0, 0.0, 0.0};
        for (int m = 0; m < 8; ++m) {
            const int32_t x = fst[8 * q + m];
            if (x < 0) continue;
            const double b = fbeta[8 * q + m];
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[c] += b * U.c[c][x];
        }
        const double den = 2.0 - fbetac[q];
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = (ubi[3 * q + c] + acc[c]) / den;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) scr[3 * q + c] = v[c];
}

}  // namespace

hipError_t fresh_enqueue_fill(ibm_grid *g, double *const uvw[3], hipStream_t s) {
    if (g->nfresh <= 0) return hipSuccess;
    const int64_t nf = g->nfresh;
    hipLaunchKernelGGL(k_fresh_fill, dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, s, nf, g->f_cell, g->f_st,
                       g->f_beta, g->f_betac, g->f_flags, g->f_ubi, cv3(uvw[0], uvw[1], uvw[2]), g->type, g->type_prev,
                       g->nx, g->ny, g->nz, g->f_scr);
    hipLaunchKernelGGL(k_ghost_scatter, dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, s, nf, g->f_cell, g->f_scr,
                       v3(uvw[0], uvw[1], uvw[2]));
    return hipGetLastError();
}

// ---- host driver ------------------------------------------------------------------------
// uvw: three device arrays (u, v, w) of N doubles, in: u^n (its ghost rows are applied in
// place, from a snapshot held in a per-ghost scratch), out: u*.  hc: three arrays, in
// H^{n-1} (ignored on the first step), out H^n.  work: the right-hand side b (0..2) and the
// second iterate buffer (3..5).
hipError_t momentum_enqueue_prep(ibm_grid *g, double *const uvw[3], double *const hc[3], double *const work[6],
                                 double dt, double a, int first, hipStream_t s) {
    const CV3 U = cv3(uvw[0], uvw[1], uvw[2]);
    hipError_t e = refresh(g, U, v3(uvw[0], uvw[1], uvw[2]), s, g->g_uscr);
    if (e != hipSuccess) return e;
    auto launch = [&](auto rpw) {
        constexpr int RPW = decltype(rpw)::value, NW = 8;
        const MTiles t = mom_tiles(g->nx, g->ny, g->nz, 128 / RPW, NW * RPW - 2, 1);
        hipLaunchKernelGGL((k_mom_rhs<RPW, NW>), dim3(t.grid), dim3(64 * NW), 0, s, mom_view(g), U,
                           v3(hc[0], hc[1], hc[2]), v3(work[0], work[1], work[2]), dt, a, first, t, g->partials);
        return t;
    };
    const MTiles t = mom_wide(g->nx) ? launch(std::integral_constant<int, 1>()) : launch(std::integral_constant<int, 2>());
    hipLaunchKernelGGL(k_mom_sum, dim3(1), dim3(256), 0, s, g->partials, t.grid, &g->sc->mom_b2);
    return hipGetLastError();
}

// one sweep from X into Y followed by the ghost rows; the residual sum of the input
// iterate lands in sc->mom_r2 when `sum` is set
hipError_t momentum_enqueue_sweep(ibm_grid *g, double *const X[3], double *const Y[3], double *const work[6],
                                  double a, double omega, bool sum, hipStream_t s) {
    const CV3 x = cv3(X[0], X[1], X[2]);
    const V3 y = v3(Y[0], Y[1], Y[2]);
    auto launch = [&](auto rpw) {
        constexpr int RPW = decltype(rpw)::value, NW = 4;
        const MTiles t = mom_tiles(g->nx, g->ny, g->nz, 128 / RPW, NW * RPW - 2, 3);
        hipLaunchKernelGGL((k_srj_sweep<RPW, NW>), dim3(t.grid), dim3(64 * NW), 0, s, mom_view(g), x, y,
                           cv3(work[0], work[1], work[2]), a, omega, t, g->partials);
        return t;
    };
    const MTiles t = mom_wide(g->nx) ? launch(std::integral_constant<int, 1>()) : launch(std::integral_constant<int, 2>());
    if (sum) hipLaunchKernelGGL(k_mom_sum, dim3(1), dim3(256), 0, s, g->partials, t.grid, &g->sc->mom_r2);
    return refresh(g, x, y, s);
}

}  // namespace ibm
