// Internal declarations of the gfx950 ghost-cell IBM projection library.
//
// Data layout in HBM (all inside the caller-owned workspace):
//   level 0 : cell type (uint8), second pressure buffer (FP64), FP32 error / residual
//             buffers for the mixed-precision path; cell fields are [nz][ny][nx].
//   metrics : 1D per-axis arrays (centres, widths, centre distances, flux coefficients),
//             so the 7-point operator of a cell is rebuilt from six scalar loads.
//   geometry: mesh, a uniform triangle bucket grid (closest-point search), per-column ray
//             crossings (classification), and the ghost list in structure-of-arrays form.
//   levels  : per coarse level the error and right-hand side, the active mask and the
//             staircase transmissibilities of each cell's three low faces, plus the
//             per-axis prolongation tables.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/ibm.h"

namespace ibm {

constexpr uint8_t T_FLUID = 0, T_GHOST = 1, T_DEAD = 2;
constexpr int GF_DEGENERATE = 1, GF_CLAMPED = 2, GF_NFALLBACK = 4, GF_SELF = 8;
constexpr int MAX_LEVELS = 24;
// Block count of the deterministic reductions: a function of the item count alone, at most
// RED_BLOCKS (enough waves to fill every SIMD); a 128^2 grid with 4096 blocks, most of them
// empty, took 9.2 us for the step's last update and 5.7 us to add up the partials.
constexpr int RED_BLOCKS = 4096;
inline int red_blocks(int64_t items, int per_block = 256) {
    const int64_t n = (items + per_block - 1) / per_block;
    return (int)(n < 1 ? 1 : n < RED_BLOCKS ? n : RED_BLOCKS);
}
// block limit of the ghost-row pass, whose partials every block of the operator pass adds up
constexpr int GHOST_ROW_BLOCKS = 1024;
constexpr int NBUCKET_MAX = 1 << 21;

// ---------------------------------------------------------------------------------------
// device views
// ---------------------------------------------------------------------------------------

template <typename T>
struct AxisCoef {  // per-axis arrays of one level
    const T *am, *ap;  // level 0: per-volume flux coefficients; unused on coarse levels
    const T *w;        // widths
};

template <typename T>
struct Fine {  // level-0 operator view in precision T
    int nx, ny, nz;
    const T *axm, *axp, *aym, *ayp, *azm, *azp;
    const T *wx, *wy, *wz;
    const uint8_t *type;
    const uint8_t *inject;  // 1: fluid cell whose prolongation has an inactive coarse contributor
};

template <typename T>
struct Coarse {  // coarse-level view in precision T
    int n[3];
    const T *w[3];        // widths
    const uint8_t *active;
    const T *Tl[3];       // transmissibility of each cell's low face (integrated form)
    T *e, *R;
    const double *mu;     // compatibility shift per unit volume (device scalar)
};

// fused red-black sweep of level 0 (sweep.hip): pout = one RB-GS sweep of pin; ev0, ev1
// (optional): events recorded when the kernel starts and when it ends
template <typename T>
hipError_t launch_sweep(const Fine<T> &F, const T *pin, T *pout, const T *f, const T *lam, hipStream_t s,
                        hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// the same FP32 sweep writing its result widened to FP64, dead cells zero
hipError_t launch_sweep_widen(const Fine<float> &F, const float *pin, double *pout, const float *f, const float *lam,
                              hipStream_t s);

// the same sweep by bricks (sweepb.hip), which launch_sweep takes for small grids
constexpr int64_t BRICK_LARGE_CELLS = 1 << 20, BRICK_LARGE_ROWS = 1 << 15;  // larger bricks from either
template <typename T, typename TO>
hipError_t launch_sweep_brick(const Fine<T> &F, const T *pin, TO *pout, const T *f, const T *lam, hipStream_t s,
                              hipEvent_t ev0, hipEvent_t ev1);

// where a coarse level's first sweep gets mu (sweepc.hip); n = 0: mu is there already
struct MuSource {
    const double *partials = nullptr;  // n sums of the restriction
    int n = 0;
    const double *vol = nullptr;
    double *mu = nullptr;
};
// red-black sweep of a coarse level (sweepc.hip): eout = one RB-GS sweep of L.e, the two buffers
// distinct; zero: L.e counts as zero and need not be read
template <typename T>
hipError_t launch_sweepC(const Coarse<T> &L, T *eout, const MuSource &ms, bool zero, hipStream_t s);
// whether a level's first sweep had better form mu from nparts partials than a launch before it
template <typename T>
bool sweepC_forms_mu(const int n[3], int nparts);
// levels that take a launch per colour instead (launch_sweepC_colours): in place, mu and the
// correction there before
bool sweepC_by_colours(const int n[3]);
template <typename T>
hipError_t launch_sweepC_colours(const Coarse<T> &L, hipStream_t s);

// fine index -> (lo, hi, weight of hi) per axis; lo is always the parent (the coarse cell
// holding the fine one)
struct ProlongTab {
    const int *lo[3], *hi[3];
    const double *t[3];
    int halved[3];  // 1: the axis is halved uniformly (fine 2I and 2I+1 make coarse I)
};

// Children of a coarse level (device): coarse index I along axis d holds the finer cells
// cs[d][I] .. cs[d][I+1]-1 (one or two).
struct ChildMap {
    const int *cs[3];
    int halved[3];  // 1: uniform halving along d
    int same[3];    // 1: nothing merged along d (cs[I] = I)
    const struct XTile *tx;  // x and z tiles of the row-wise restrictions, one more at the end
    const struct ZTile *tz;
    int ntx, ntz;
};
struct XTile {
    int I0, i0;  // first coarse column and its first child
};
struct ZTile {
    int K0, k0;     // first coarse plane and its first child
    uint64_t ends;  // bit k: finer plane k0 + k is the last of a coarse plane.  (A march that looks the
                    // next end up as it goes waits for that load, and so for the plane loads before it.)
};

// z-march passes of level 0 (finepass.hip).  The reductions write one partial per
// workgroup; *nparts receives their count (at most zmarch_partials_max).
template <typename T>
hipError_t launch_restrict0(const Fine<T> &F, const T *p, const T *f, const T *lam, const Coarse<T> &C,
                            const ChildMap &M, double *partials, int *nparts, hipStream_t s);
template <typename T>
hipError_t launch_prolong0(const Fine<T> &F, const T *pcur, T *pnext, const Coarse<T> &C, const ProlongTab &P,
                           hipStream_t s);
// Krylov operator on fluid rows; w is 0 on dead cells and not written on ghost cells.  dots 1
// and 2: w = S y - mu, sums of o w and of w w per workgroup (stride 2).  dots 3: the residual
// w = o - S y (o the right-hand side; mu unused), sum V w per workgroup.
// mu, the image's volume-weighted fluid mean: the sum of n partials over the fluid volume
struct MeanParts {
    const double *part;
    int n;
    const double *vol;
};
hipError_t launch_apply_fluid(const Fine<double> &F, const double *y, double *w, const double *o, const MeanParts &mu,
                              int dots, double *partials, int *nparts, hipStream_t s);
hipError_t launch_jacobi0(const Fine<double> &F, const double *y, const double *f, double *out, double omega,
                          hipStream_t s);
int64_t zmarch_partials_max(int nx, int ny, int nz);

// Tiling of the row-wise restrictions: a workgroup of 64 RM_W threads takes, a wave per coarse row,
// the coarse columns that start in a window of RM_FX finer ones, RM_W coarse rows and the coarse
// planes that start in a window of finer ones, tile by tile in a grid-stride loop; the grid is a
// multiple of 8, at most the tile count rounded up and at most cap (a multiple of 8).
// A window's coarse columns span at most RM_FX + 1 finer ones, which with one more on either side
// fill a wave however few of them are merged (32 coarse columns left 24 of 64 lanes idle on
// a level of 160 x 100 x 99 cells).
constexpr int RM_FX = 61, RM_W = 4, RM_NT = 64 * RM_W;
// The z tiles are windows of finer planes too, so that a tile's work does not depend on how many
// planes are merged where it lies: each XCD takes a contiguous range of tiles, and with tiles of
// equal coarse planes those in the middle of a stretched grid had the most (384^3: 343 us, by
// windows 317).
// Their size minimises rounds of resident workgroups x (planes + RM_ZCOST), a tile's two planes
// shared with its neighbours and its start counting as RM_ZCOST planes: a round that is not full
// costs as much as one that is (wing, 2.3 rounds 33 us, one of longer tiles 25.5).
constexpr int RM_RESIDENT = 4, RM_ZCOST = 3, RM_ZMAX = 60;  // workgroups per CU; ZTile::ends has 64 bits
struct RowTiles {
    int ntx, nty, ntiles;
};
hipError_t row_tiles(const ChildMap &M, const int cn[3], int64_t cap, RowTiles *t, int *grid);

struct GhostView {
    int64_t ng;
    const int32_t *cell;
    const int32_t *st;      // 8 per ghost, -1 = unused / own Neumann slot
    const uint8_t *gmask;   // bit m: member m is a ghost cell
    const double *beta;     // 8 per ghost
    const double *h;        // right-hand side of the ghost equation
    const int32_t *flags;
};

// reduction scratch shared by the solver kernels (device)
struct Scalars {
    double lambda;      // current uniform source shift
    double delta;       // lambda_{k+1} - lambda_k (mixed path: FP64)
    float delta32;      // same, FP32 (inner right-hand side shift)
    float pad0;
    double norm;        // ||r - lambda||_2 after the last norm pass
    double rel;         // norm / ref
    double ref;         // reference norm ||f - Vmean(f)||
    double vmean;       // scratch mean
    double div_max;
    double ghost_res;   // max ghost-equation residual of the returned pressure
    int bad;            // non-finite seen
    int pad1;
    // Krylov (BiCGStab) scalars
    double rho, rho_old, alpha, omega, beta;
    double mu_v;        // volume-weighted fluid mean removed from a residual
    double zero;        // constant 0 (shift of the preconditioner's right-hand side)
    float zero32, pad2;
    double rh2;         // squared norm of the shadow residual (set when it is (re)started)
    int brk;            // near-breakdown seen in the last step: the host restarts the shadow residual
    int pad3;
    double mu[MAX_LEVELS];
    double vol[MAX_LEVELS];   // summed volume of the active cells of each level
    double mom_b2;            // advection-diffusion step: sum of b^2 over fluid rows
    double mom_r2;            // sum of r^2 at the input of the last sweep
};

// ---------------------------------------------------------------------------------------
// host-side state
// ---------------------------------------------------------------------------------------

struct LevelHost {
    int n[3];
    int halved[3];  // uniform halving relative to the next finer level (see plan_levels)
    int same[3];    // nothing merged relative to the next finer level
    std::vector<double> f[3], c[3], w[3];
    std::vector<int> cs[3];  // children starts in the next finer level (levels >= 1)
    int *cs_d[3] = {nullptr, nullptr, nullptr};  // device copy of cs
    std::vector<XTile> tx;  // tiles of the restriction into this level (see ChildMap)
    std::vector<ZTile> tz;
    XTile *tx_d = nullptr;
    ZTile *tz_d = nullptr;
    int64_t ncell() const { return (int64_t)n[0] * n[1] * n[2]; }
    // device
    uint8_t *active = nullptr;
    double *T64[3] = {nullptr, nullptr, nullptr};
    float *T32[3] = {nullptr, nullptr, nullptr};
    double *w64[3] = {nullptr, nullptr, nullptr};
    float *w32[3] = {nullptr, nullptr, nullptr};
    double *c64[3] = {nullptr, nullptr, nullptr};
    double *e64 = nullptr, *R64 = nullptr;
    float *e32 = nullptr, *R32 = nullptr;
    // second error buffer of the out-of-place coarse sweep (levels of more than SMALL_LEVEL
    // cells); swapped with e after each sweep
    double *e64b = nullptr;
    float *e32b = nullptr;
    // prolongation tables of THIS level from the next coarser one
    int *plo[3] = {nullptr, nullptr, nullptr}, *phi[3] = {nullptr, nullptr, nullptr};
    // every halved axis: the second contributor of cell 2I is I-1 and of 2I+1 is I+1 (or none
    // at a wall), which the fully halved prolongation kernel relies on (checked on the host
    // with the arithmetic the device tables use)
    bool prolong_sides = false;
    double *pt[3] = {nullptr, nullptr, nullptr};
    double vol_active = 0.0;  // device-computed, copied back at hierarchy build
};

// the levels that one workgroup takes to the bottom of the V-cycle (tail.hip): the first has at
// most SMALL_LEVEL cells, the others together take at most TAIL_E - SMALL_LEVEL table entries
constexpr int SMALL_CPT = 4, SMALL_LEVEL = 1024 * SMALL_CPT;
constexpr int TAIL_MAX = 8, TAIL_E = 2 * SMALL_LEVEL;
struct TailTables {  // per cell of those levels, rebuilt with the hierarchy
    double *c64 = nullptr;     // 8 x TAIL_E coefficients
    float *c32 = nullptr;
    double *w = nullptr;       // 3 x TAIL_E prolongation weights
    uint2 *meta = nullptr;     // TAIL_E
    uint32_t *down = nullptr;  // TAIL_E
};
int tail_first(const LevelHost *lev, int nlev);  // the first such level; nlev: none
hipError_t launch_tail_tables(ibm_grid *g, hipStream_t s);
template <typename T>
hipError_t launch_tail(ibm_grid *g, int lt, const Coarse<T> &first, int nparts, const ibm_solve_opts *o, hipStream_t s);

enum Stage { ST_CREATED = 0, ST_BOUND = 1, ST_GEOMETRY = 2, ST_CLASSIFIED = 3, ST_STENCILS = 4 };

struct SolveState {  // in-flight solve of the step API
    bool active = false, done = true;
    const double *rhs = nullptr;
    double *p_user = nullptr;
    ibm_solve_opts o{};
    hipStream_t stream = nullptr;
    int cycles = 0, status = 0;
    int pending = 0;            // cycles enqueued since the last poll read
    double r0 = 0.0;
    hipEvent_t ev = nullptr;
    bool ev_pending = false;
    int cur = 0;                // which buffer holds the iterate (0 = user p, 1 = workspace)
    bool finishing = false;     // gauge enqueued, waiting for its event
    int phase = 0;              // BiCGStab: 1 while a true-residual confirmation is in flight
    int restarts = 0;           // BiCGStab restarts after a near-breakdown
    double t0 = 0.0;
};

// optional per-launch timing of the level-0 smoother (HIP events on the launch stream)
struct Prof {
    bool on = false;
    int stride = 1;              // time every stride-th level-0 sweep
    long long seq = 0;           // level-0 sweeps launched since profiling was switched on
    std::vector<hipEvent_t> ev;  // start/stop pairs
    std::vector<int> kind;       // per pair: 0 FP64 sweep, 1 FP32 sweep
    int used = 0;
    double ms[2] = {0.0, 0.0};
    long long count[2] = {0, 0};
};

}  // namespace ibm

struct ibm_grid {
    hipEvent_t ev_read = nullptr;  // the residual's copy to the host
    int nx, ny, nz;
    int64_t N;
    std::vector<double> xf, yf, zf;
    int stage = ibm::ST_CREATED;
    std::string err;
    // workspace
    char *ws = nullptr;
    size_t ws_bytes = 0;
    int64_t nv_max = 0, nt_max = 0, ghost_max = 0;
    ibm_precision prec = IBM_FP64;
    int device = 0;
    // level-0 device arrays
    uint8_t *type = nullptr;
    uint8_t *inject0 = nullptr;            // per cell: prolongation falls back to injection
    double *p2 = nullptr;                  // second FP64 pressure buffer
    double *frhs = nullptr;                // projection right-hand side
    float *e32a = nullptr, *e32b = nullptr, *r32 = nullptr;
    // start iterate of the Krylov preconditioner's V-cycle: zero except at the ghost cells,
    // whose values are written before each use (cleared whenever the ghost list is rebuilt)
    double *pz = nullptr;
    float *pz32 = nullptr;
    double *faces[3] = {nullptr, nullptr, nullptr};
    double *c0[3] = {nullptr, nullptr, nullptr}, *w0[3] = {nullptr, nullptr, nullptr};
    double *dc0[3] = {nullptr, nullptr, nullptr};
    double *am0[3] = {nullptr, nullptr, nullptr}, *ap0[3] = {nullptr, nullptr, nullptr};
    float *am0f[3] = {nullptr, nullptr, nullptr}, *ap0f[3] = {nullptr, nullptr, nullptr};
    float *w0f[3] = {nullptr, nullptr, nullptr};
    // mesh and geometry scratch
    int64_t nv = 0, nt = 0;
    double *verts = nullptr, *verts_in = nullptr;  // the mesh in use, and the one being checked
    int32_t *tris = nullptr, *tris_in = nullptr;   // (exchanged when it is accepted)
    int32_t *bucket_off = nullptr, *bucket_cnt = nullptr, *bucket_ent = nullptr;
    int nb[3] = {1, 1, 1};
    double bmin[3] = {0, 0, 0}, bsize[3] = {1, 1, 1};
    double bext[3] = {0, 0, 0};  // largest triangle extent per axis (padded for rounding)
    int32_t *col_cnt = nullptr, *col_off = nullptr, *col_fill = nullptr;
    double *crossings = nullptr;
    int64_t cross_cap = 0;
    int32_t *blk_cnt = nullptr;            // per-block counts for compaction / scans
    int64_t *counters = nullptr;           // device counters (fluid, ghost, dead, odd, overflow...)
    // ghosts
    int64_t ng = 0;
    int64_t ndegenerate = 0;
    int32_t *g_cell = nullptr, *g_st = nullptr, *g_flags = nullptr, *g_tri = nullptr;
    uint8_t *g_mask = nullptr;
    double *g_bi = nullptr, *g_n = nullptr, *g_ip = nullptr, *g_beta = nullptr, *g_betag = nullptr;
    double *g_dl = nullptr, *g_h = nullptr, *g_data = nullptr;
    double *g_scale = nullptr;             // diagonal of the flux stencil at each ghost cell
    double *g_rhs = nullptr;               // ghost right-hand sides of a preconditioner call
    double *g_betaD = nullptr;             // 8 per ghost: Dirichlet (velocity) weights
    double *g_betaDg = nullptr;            // per ghost: weight of the intercept value
    double *g_ubi = nullptr;               // 3 per ghost: velocity at the body intercept
    double *g_uscr = nullptr;              // 3 per ghost: held-back ghost values of an in-place pass
    std::vector<int32_t> topo_tris;        // triangles of the last accepted mesh, if few, on the host
    int64_t topo_nv = 0;                   // and its vertex count
    // fresh cells of the last move (capacity ghost_max)
    uint8_t *type_prev = nullptr;          // cell types before the move
    int64_t nfresh = 0;
    int32_t *f_cell = nullptr, *f_tri = nullptr, *f_st = nullptr, *f_flags = nullptr;
    double *f_bi = nullptr, *f_ip = nullptr, *f_beta = nullptr, *f_betac = nullptr, *f_ubi = nullptr,
           *f_scr = nullptr;
    double diag_max = -1.0;                // max over cells of the flux-coefficient sum (< 0: not read yet)
    double t_setup = 0.0;                  // seconds of the last set_geometry + classify + stencils
    std::vector<double> srj_omega;         // relaxation factors of the scheduled-Jacobi preconditioner
    // Krylov vectors (FP64, full grid)
    double *kv[10] = {nullptr};
    // multigrid
    int nlev = 0;
    ibm::LevelHost lev[ibm::MAX_LEVELS];
    ibm::TailTables tail;
    double *partials = nullptr;            // RED_BLOCKS * 4 doubles
    ibm::Scalars *sc = nullptr;            // device scalars
    ibm::Scalars *sc_host = nullptr;       // pinned host mirror
    int64_t nfluid = 0, nghost_cells = 0, ndead = 0;
    double vol_fluid = 0.0;
    ibm::SolveState ss;
    ibm::Prof prof;
    // debug: fill every floating-point sub-buffer of the workspace with NaN at bind time
    // (ibm_debug_poison), so a value read before the library wrote it shows up
    bool debug_poison = false;
};

namespace ibm {

// workspace planner: computes offsets (base == nullptr -> sizing only)
// Large arrays start STAGGER further off the 4 KB grid each: fields of 2^24 doubles and the like lie
// a large power of two apart otherwise, and the streams of a pass meet in the same channels (384^3:
// fine sweep 340 -> 331 us, operator 315 -> 302; steps of 140 KB and 1 MB gave the same).
constexpr int64_t STAGGER_MIN = 1 << 20;
constexpr size_t STAGGER = 4096 + 256;
struct Plan {
    size_t off = 0;
    size_t large = 0;
    char *base = nullptr;
    // optional: (offset, bytes) of every floating-point sub-buffer, for the poisoned bind
    std::vector<std::pair<size_t, size_t>> *fp_spans = nullptr;
    template <typename T>
    T *take(int64_t count) {
        off = (off + 255) & ~size_t(255);
        if (count >= STAGGER_MIN) off += STAGGER * (large++ % 16);
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        const size_t bytes = sizeof(T) * (size_t)(count > 0 ? count : 1);
        if (fp_spans && std::is_floating_point<T>::value) fp_spans->emplace_back(off, bytes);
        off += bytes;
        return p;
    }
};

// hierarchy plan on the host (dims + coarse faces), same rule for sizing and binding
// the level's child map (device pointers; level >= 1)
ChildMap child_map(const LevelHost &C);
void plan_levels(int nx, int ny, int nz, const double *xf, const double *yf, const double *zf,
                 LevelHost *lev, int *nlev);
size_t layout(ibm_grid *g, Plan &P, int nx, int ny, int nz, int64_t nv_max, int64_t nt_max, int64_t gmax,
              ibm_precision prec, LevelHost *lev, int nlev);

// classification buffers (geometry.hip): a handle's workspace or the static scratch of the
// no-allocation entry point
struct ClassifyBufs {
    int nx, ny, nz;
    const double *verts;
    const int32_t *tris;
    int64_t nt;
    const double *xc, *yc, *zc;           // cell centres per axis
    int32_t *col_cnt, *col_off, *col_fill;  // ncol + 1 each
    double *crossings;
    int64_t cross_cap;
    int64_t *counters;                    // 8
    int64_t *blk;                         // classify_scan_blocks(ncol + 1)
    int64_t *mark_parts;                  // classify_mark16_parts(nx, ny, nz)
    uint8_t *type;
};
hipError_t launch_classify_cells(const ClassifyBufs &B, hipStream_t s);
int64_t classify_mark16_parts(int nx, int ny, int nz);
int64_t classify_scan_blocks(int64_t n);

// error reporting shared by the entry points (api.hip): sets the thread's last error
ibm_status report_error(ibm_status st, const std::string &msg);

// kernel launchers (geometry.hip)
hipError_t launch_metrics(ibm_grid *g, hipStream_t s);
hipError_t launch_buckets(ibm_grid *g, hipStream_t s);
// check and extents of an uploaded mesh (device arrays); synchronises the stream
constexpr int MESH_BAD_VERT = 1, MESH_BAD_INDEX = 2, MESH_BAD_TOPO = 4;
constexpr int64_t MESH_TAB_PAD = 64;  // slots of the edge table beyond 3 per triangle
struct MeshScan {
    double lo[3], hi[3], ext[3];  // over the triangles with valid indices
    int bad;
};
hipError_t launch_mesh_scan(ibm_grid *g, const double *V, int64_t nv, const int32_t *T, int64_t nt, MeshScan *out,
                            hipStream_t s);
hipError_t launch_classify(ibm_grid *g, hipStream_t s, int64_t counts[4]);
hipError_t launch_stencils(ibm_grid *g, hipStream_t s);
hipError_t launch_ghost_h(ibm_grid *g, hipStream_t s);
hipError_t launch_hierarchy(ibm_grid *g, hipStream_t s);
hipError_t launch_fresh(ibm_grid *g, hipStream_t s, int64_t *nfresh);

// solver launchers (solver.hip)
hipError_t sweep0_f64(ibm_grid *g, const double *pin, double *pout, const double *f, const double *lambda,
                      hipStream_t s);
hipError_t refresh_f64(ibm_grid *g, const double *src_ghost, double *dst, hipStream_t s);
hipError_t apply0_f64(ibm_grid *g, const double *p, double *out, hipStream_t s);
// swept: vcycle_ahead, the cycle's first pre-smoothing sweep and ghost refresh, is done
hipError_t vcycle_f64(ibm_grid *g, double **bufs, int *cur, const double *f, hipStream_t s, const ibm_solve_opts *o,
                      bool swept = false);
hipError_t vcycle_ahead(ibm_grid *g, double **bufs, int *cur, const double *f, hipStream_t s);
hipError_t vcycle_mixed(ibm_grid *g, double **bufs, int *cur, const double *f, hipStream_t s,
                        const ibm_solve_opts *o);
hipError_t norm_pass(ibm_grid *g, const double *p, const double *f, hipStream_t s, bool write_r32, bool first);
hipError_t ref_norm_pass(ibm_grid *g, const double *f, hipStream_t s);
hipError_t gauge_pass(ibm_grid *g, const double *pcur, double *pdst, hipStream_t s);
hipError_t ghost_residual_pass(ibm_grid *g, const double *p, hipStream_t s);
hipError_t rhs_pass(ibm_grid *g, const double *u, const double *v, const double *w, double dt, double *f,
                    hipStream_t s);
hipError_t cell_to_faces_pass(ibm_grid *g, const double *u, const double *v, const double *w, double *uf,
                              double *vf, double *wf, hipStream_t s);
hipError_t correct_cells_pass(ibm_grid *g, double *u, double *v, double *w, const double *p, double dt,
                              hipStream_t s);
hipError_t correct_pass(ibm_grid *g, double *u, double *v, double *w, const double *p, double dt,
                        hipStream_t s);
hipError_t divmax_pass(ibm_grid *g, const double *u, const double *v, const double *w, hipStream_t s);
hipError_t init_solution(ibm_grid *g, double *p, double *p2, int use_guess, hipStream_t s);
hipError_t krylov_setup(ibm_grid *g, hipStream_t s);
hipError_t krylov_residual(ibm_grid *g, const double *f, const double *x, hipStream_t s);
// what of a step is enqueued before the host has seen the residual of the one before
enum Ahead { AHEAD_NONE, AHEAD_P, AHEAD_SWEEP };
// first: the first step after krylov_residual of a new solve (p and v are not read)
hipError_t krylov_step(ibm_grid *g, double *x, const ibm_solve_opts *o, bool first, hipStream_t s,
                       Ahead done = AHEAD_NONE);
hipError_t krylov_ahead(ibm_grid *g, const ibm_solve_opts *o, bool first, Ahead what, hipStream_t s);
// the handle's last geometry set-up time is g->t_setup (seconds, host wall clock)
hipError_t krylov_restart(ibm_grid *g, hipStream_t s);

// advection-diffusion half-step launchers (momentum.hip)
hipError_t momentum_enqueue_prep(ibm_grid *g, double *const uvw[3], double *const hc[3], double *const work[6],
                                 double dt, double a, int first, hipStream_t s);
hipError_t momentum_enqueue_sweep(ibm_grid *g, double *const X[3], double *const Y[3], double *const work[6],
                                  double a, double omega, bool sum, hipStream_t s);
hipError_t fresh_enqueue_fill(ibm_grid *g, double *const uvw[3], hipStream_t s);

}  // namespace ibm
