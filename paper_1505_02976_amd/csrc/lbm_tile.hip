// Several time steps per launch: a block keeps a tile of nodes in LDS.
//
// Small grids are bound by latency, not by memory or arithmetic: a step of 128 x 128 nodes
// is 256 wavefronts on 1024 SIMDs, so what a step costs is the launches (about 4 us each
// with their kernel's start and end), the events between the two streams of a two-step pass
// and the serial walk of its wavefronts.  Here one launch advances the whole grid by ns
// steps.  A block owns a rectangular tile and starts from its nodes and ns - 1 more on every
// side; step s computes the nodes within ns - s of the tile (fewer each step; a side that is
// a wall of the grid does not shrink), one per thread, the first step pulling from the source
// buffer, the later ones from LDS, where every step leaves its post-collision populations as
// the one-step path would store them.  Tiles recompute their overlap; no block waits for
// another.  Every node update is the one-step node code with the same inputs, so ns steps
// here are bitwise ns single steps.
//
// A wall node pulls at its reference node x_f and shares the state computation with the
// other nodes, so that a wall wavefront adds only the boundary scheme to its chain.  The
// scheme reaches three nodes inward (x_f, x_ff and their pulls), which the tile holds: tiles
// are at least four nodes wide wherever there is more than one.
//
// Blocks are dealt to the XCDs in contiguous ranges (xcd_block), so that neighbouring tiles,
// whose halos share cache lines, share an L2: without it a 250 x 250 FP32 launch of one step
// took 10.1 us instead of 6.7.
//
// Measured (one step, 100-step calls, two-step passes before): 128 x 128 FP64 27 -> 2.8 us,
// 250 x 250 FP32 22 -> 3.1 us, 500 x 500 FP32 25 -> 7.3 us, 1350 x 1350 FP32 45 -> 36 us; a
// grid of at most 512 nodes (one block, any number of steps per launch) 17 -> 1.7 us.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "lbm_tile.h"

namespace lbm {

constexpr int TILE_NT = 512;      // nodes of the largest region, threads of the largest block

// Stored value in LDS (what the one-step path would store).
__device__ __forceinline__ void lds_put(double *p, double v, float) { *p = v; }
__device__ __forceinline__ void lds_put(float *p, float v, float) { *p = v; }
__device__ __forceinline__ void lds_put(__half *p, float v, float scale) { *p = __float2half(v * scale); }

// Region of a tile: the nodes of the launch's first step.
struct TileRegion {
    int X0, X1, Y0, Y1;              // the tile (written by this block)
    int xlo, xhi, ylo, yhi;
    bool oxl, oxh, oyl, oyh;         // sides that shrink by one node per step
    bool walls;                      // holds a wall node
};

__device__ __forceinline__ TileRegion tile_region(const KParams &P, const TileGrid &g, int b, int ns)
{
    TileRegion t;
    const int ty = tile_row(g, b), tx = b - ty * g.nbx;
    t.X0 = tx * g.tw + min(tx, g.rx); t.X1 = t.X0 + g.tw + (tx < g.rx ? 1 : 0);
    t.Y0 = ty * g.th + min(ty, g.ry); t.Y1 = t.Y0 + g.th + (ty < g.ry ? 1 : 0);
    t.xlo = t.X0 - (ns - 1); t.xhi = t.X1 + (ns - 1); t.ylo = t.Y0 - (ns - 1); t.yhi = t.Y1 + (ns - 1);
    t.oxl = t.oxh = t.oyl = t.oyh = true;
    if (g.nbx == 1 || (!P.px && t.xlo <= 0)) { t.xlo = 0; t.oxl = false; }
    if (g.nbx == 1 || (!P.px && t.xhi >= P.nx)) { t.xhi = P.nx; t.oxh = false; }
    if (g.nby == 1 || (!P.py && t.ylo <= 0)) { t.ylo = 0; t.oyl = false; }
    if (g.nby == 1 || (!P.py && t.yhi >= P.ny)) { t.yhi = P.ny; t.oyh = false; }
    t.walls = (!P.px && (!t.oxl || !t.oxh)) || (!P.py && (!t.oyl || !t.oyh));
    return t;
}

// The coefficients at a node's porosity for one step.  AGAIN: formed in every step from the few
// that EpsK keeps (three operations), where registers are short; held across the steps otherwise
// (the adjoint's forward states at 256 x 256 FP32: 3 % faster).
template <bool AGAIN, typename R> __device__ __forceinline__ EpsC<R> eps_step(KConst pc, EpsK<R> &h)
{
    if (AGAIN) asm volatile("" : "+v"(h.eps), "+v"(h.c1));
    return eps_from<R>(pc->nu_over_K, h);
}

// ns steps of one tile.  lds: 18 planes of TILE_NT values, [q][node of the region].  WALLS: the
// region holds wall nodes.  WRAP: it spans the grid along a periodic direction (wx, wy),
// whose pulls wrap inside it.  hist != 0: every step s is stored, at dst + (s - 1) hist.
template <typename S, bool FIELD, bool DENSE, bool WALLS, bool WRAP>
__device__ __forceinline__ void tile_steps(const S *__restrict__ src, S *__restrict__ dst, const KParams &P,
                                           KConst Pc, const TileRegion &t, bool wx, bool wy, int ns, long long hist,
                                           S *__restrict__ lds)
{
    using R = typename Prec<S>::R;
    const int rw = t.xhi - t.xlo, rh = t.yhi - t.ylo;
    // threadIdx.x / rw (exact: the quotient is at least 1 / (2 rw) away from the next integer)
    const int ly = (int)(((float)threadIdx.x + 0.5f) * __builtin_amdgcn_rcpf((float)rw)), lx = (int)threadIdx.x - ly * rw;
    int x = t.xlo + lx, y = t.ylo + ly;
    const bool own = ly < rh && x >= t.X0 && x < t.X1 && y >= t.Y0 && y < t.Y1;
    if (P.px) x = ((x % P.nx) + P.nx) % P.nx;
    if (P.py) y = ((y % P.ny) + P.ny) % P.ny;
    // the last step the node takes: all for the block's own nodes, one less per node of
    // distance from the tile towards a side that shrinks (0: no node of the region)
    int last = ns;
    if (!own) {
        last = ns - 1;
        if (t.oxl) last = min(last, lx + 1);
        if (t.oxh) last = min(last, rw - lx);
        if (t.oyl) last = min(last, ly + 1);
        if (t.oyh) last = min(last, rh - ly);
        if (ly >= rh) last = 0;
    }
    WallInfo w = {-1, -1, 0, 0};
    if (WALLS) w = wall_info(P, x, y);
    const bool wall = WALLS && (w.xw >= 0 || w.yw >= 0);
    const int xr = x + w.dx, yr = y + w.dy;               // where the node pulls: itself, or x_f
    const int nff = w.dx + w.dy * rw;                     // from the node to x_f, and to x_ff from there
    S *const L = lds + (ly * rw + lx);
    const S *const r0 = L + nff;
    // steps to the columns x -+ 1 and rows y -+ 1 of the node it pulls at
    const int lxr = lx + w.dx, lyr = ly + w.dy;
    const int cm = WRAP && wx && lxr == 0 ? rw - 1 : -1, cp = WRAP && wx && lxr == rw - 1 ? 1 - rw : 1;
    const int rm = WRAP && wy && lyr == 0 ? (rh - 1) * rw : -rw, rp = WRAP && wy && lyr == rh - 1 ? (1 - rh) * rw : rw;
    EpsK<R> hr, ho;                                       // at the pulled node, at the node itself
    constexpr bool TAB = DENSE && WALLS;
    __shared__ WallC<R> wtab[TAB ? 9 : 1];                // of the four walls and the four corners
    const int wi = TAB ? (w.dx + 1) + 3 * (w.dy + 1) : 0;
    WallC<R> wc = {};
    bool neumann = false;
    R f[9], g[9], Tdff = R(0);
    if (last > 0) {
        if (FIELD) hr = ho = eps_keep<R>(P, eps_value(P, xr, yr));
        if (wall) {
            wc = wall_consts<R>(P, w);
            if (TAB) wtab[wi] = wc;
            neumann = !wc.iso;
            if (FIELD) ho = eps_keep<R>(P, eps_value(P, x, y));
        }
    }
    if (TAB) __syncthreads();
    if (last > 0) {
        gather<S, R>(src, P, xr, yr, f, g);
        if (neumann) Tdff = gather_Td<S, R>(src, P, cst<R>(P), x + 2 * w.dx, y + 2 * w.dy);
    }
    const int store_from = hist ? 1 : ns;
#pragma clang loop unroll(disable)
    for (int s = 1;; ++s) {
        const KConst pc = fresh(Pc);
        Cst<R> k;
        load_consts(pc, k);
        const R T0 = R(pc->T0);
        const float hinv = pc->hinv, hscale = pc->hscale;
        EpsC<R> er, eo;
        if (FIELD) {
            er = eps_step<DENSE, R>(pc, hr);
            eo = WALLS ? eps_step<DENSE, R>(pc, ho) : er;
        } else {
            load_eps(pc, er);
            eo = er;
        }
        if (s <= last) {
            Macro<R> m;
            node_macro_full<R>(f, g, T0, k, er, m);
            if (wall) {
                Macro<R> mb;
                if (TAB) {
                    wc = wtab[wi];
                    __builtin_amdgcn_sched_barrier(0);    // not ahead of the state, which fills the registers
                }
                wall_from_state<R>(T0, k, wc, er, eo, m, f, g, Tdff, f, g, mb);
                if (TAB) __builtin_amdgcn_sched_barrier(0);
                m = mb;
            }
            node_collide<R>(f, g, m, T0, k, WALLS ? eo : er);
            if (own && s >= store_from) store_node<S, R>(dst + (s - 1) * hist, P, x, y, f, g);
        }
        if (s == ns) break;
        if (s <= last) {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                lds_put(L + i * TILE_NT, f[i], hscale);
                lds_put(L + (9 + i) * TILE_NT, g[i], hscale);
            }
        }
        __syncthreads();
        if (s < last) {
            const S *const qm = r0 + rm, *const qp = r0 + rp;
            const S *const b[9] = {r0, r0 + cm, qm, r0 + cp, qp, qm + cm, qm + cp, qp + cp, qp + cm};
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                f[i] = R(Store<S>::ld(b[i] + i * TILE_NT, hinv));
                g[i] = R(Store<S>::ld(b[i] + (9 + i) * TILE_NT, hinv));
            }
            if (neumann) {
                R sg = R(0);
#pragma unroll
                for (int i = 0; i < 9; ++i) sg += R(Store<S>::ld(b[i] + nff + (9 + i) * TILE_NT, hinv));
                Tdff = (sg + k.halfQ) * k.isig;
            }
        }
        __syncthreads();
    }
}

template <typename S, bool FIELD, bool DENSE>
__device__ __forceinline__ void tile_block(const S *__restrict__ src, S *__restrict__ dst, const KParams &P, KConst Pc,
                                           const TileGrid &g, int b, int ns, long long hist, S *__restrict__ lds)
{
    const TileRegion t = tile_region(P, g, b, ns);
    const bool wx = P.px && g.nbx == 1, wy = P.py && g.nby == 1;
    if (wx || wy) tile_steps<S, FIELD, DENSE, true, true>(src, dst, P, Pc, t, wx, wy, ns, hist, lds);
    else if (t.walls) tile_steps<S, FIELD, DENSE, true, false>(src, dst, P, Pc, t, wx, wy, ns, hist, lds);
    else tile_steps<S, FIELD, DENSE, false, false>(src, dst, P, Pc, t, wx, wy, ns, hist, lds);
}

// Wavefronts per SIMD that the kernels leave room for: four, except in FP64 off the dense
// variant, whose wall tiles hold up to 226 registers.  FP32 and FP16 with a porosity field took 138
// without the bound and ran three: 300 x 300 FP32 5.0 us per step against 4.0, 700 x 800 FP16 19.0
// against 15.5.
template <typename S, bool DENSE> struct TileWaves { static constexpr int v = sizeof(S) != 8 || DENSE ? 4 : 1; };

// P is the third parameter: it starts 16 bytes into the kernel's parameter segment.
template <typename S, bool FIELD, bool DENSE>
__global__ void __launch_bounds__(TILE_NT, (TileWaves<S, DENSE>::v))
k_tile(const S *__restrict__ src, S *__restrict__ dst, KParams P, TileGrid g, int ns, long long hist)
{
    __shared__ S lds[18 * TILE_NT];
    const KConst Pc = (KConst)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + 16);
    tile_block<S, FIELD, DENSE>(src, dst, P, Pc, g, xcd_block(blockIdx.x, gridDim.x), ns, hist, lds);
}

// Batched: item (problem, tile).  FIELDS: no problem, all, or some have a porosity field.  Those of
// uniform porosity take the host's coefficients, as alone (the device's of the same porosity differ
// in the last bit).  The item, and with it the problem's parameters, are wavefront-uniform.
template <typename S, int FIELDS, bool DENSE>
__global__ void __launch_bounds__(TILE_NT, (TileWaves<S, DENSE>::v))
k_batch_tile(const BatchProblem *__restrict__ probs, const int2 *__restrict__ items, int parity, int ns)
{
    __shared__ S lds[18 * TILE_NT];
    const int2 it = items[xcd_block(blockIdx.x, gridDim.x)];
    const BatchProblem &B = probs[__builtin_amdgcn_readfirstlane(it.x)];
    const S *const src = static_cast<const S *>(B.buf[parity]);
    S *const dst = static_cast<S *>(B.buf[parity ^ 1]);
    const int b = __builtin_amdgcn_readfirstlane(it.y);
    if (FIELDS == FIELDS_ALL || (FIELDS == FIELDS_SOME && B.P.field))
        tile_block<S, true, DENSE>(src, dst, B.P, (KConst)&B.P, B.tile, b, ns, 0, lds);
    else
        tile_block<S, false, DENSE>(src, dst, B.P, (KConst)&B.P, B.tile, b, ns, 0, lds);
}

// The dense variant (DENSE, FP64) fits four wavefronts per SIMD instead of two: its wall tiles
// spill and read the wall constants from LDS when they need them, which other blocks hide once
// there are several rounds of them.  us per step without and with it: 1025 x 1025 45.4 and 37.1,
// 1200 x 1100 55.2 and 44.9, 1537 x 1025 with a porosity field 66 and 57; but 800 x 700 with a field
// 24.5 and 24.8, 600 x 500 17.5 and 21.2, 128 x 128 2.82 and 3.0.
constexpr long long TILE_DENSE = 700000;
static bool tile_dense(int storage, long long nodes) { return storage == 0 && nodes >= TILE_DENSE; }

// Largest region of a launch of ns steps: its width and height.
static void tile_extent(const TileGrid &g, int ns, int &w, int &h)
{
    w = g.tw + (g.rx ? 1 : 0) + (g.nbx > 1 ? 2 * (ns - 1) : 0);
    h = g.th + (g.ry ? 1 : 0) + (g.nby > 1 ? 2 * (ns - 1) : 0);
}

template <typename S>
static hipError_t tile_t(const void *src, void *dst, const KParams &P, const TileGrid &g, int ns, long long hist,
                         hipStream_t st)
{
    const dim3 grid(g.nbx * g.nby), block(tile_threads(g, ns));
    const auto dense = P.field ? &k_tile<S, true, sizeof(S) == 8> : &k_tile<S, false, sizeof(S) == 8>;
    const auto sparse = P.field ? &k_tile<S, true, false> : &k_tile<S, false, false>;
    const auto k = tile_dense(sizeof(S) == 8 ? 0 : 1, (long long)P.nx * P.ny) ? dense : sparse;
    hipLaunchKernelGGL(k, grid, block, 0, st, (const S *)src, (S *)dst, P, g, ns, hist);
    return hipGetLastError();
}

hipError_t launch_tile(int storage, const void *src, void *dst, const KParams &P, const TileGrid &g, int ns,
                       long long hist, hipStream_t st)
{
    if (ns < 1 || tile_threads(g, ns) > TILE_NT) return hipErrorInvalidValue;
    switch (storage) {
    case 0: return tile_t<double>(src, dst, P, g, ns, hist, st);
    case 1: return tile_t<float>(src, dst, P, g, ns, hist, st);
    case 2: return tile_t<__half>(src, dst, P, g, ns, hist, st);
    default: return hipErrorInvalidValue;
    }
}

template <typename S>
static hipError_t batch_tile_t(const BatchProblem *probs, const int2 *items, int nitems, int fields, long long nodes,
                               int threads, int parity, int ns, hipStream_t st)
{
    constexpr bool D = sizeof(S) == 8;
    const bool d = tile_dense(D ? 0 : 1, nodes);
    const auto k = fields == FIELDS_NONE ? (d ? &k_batch_tile<S, FIELDS_NONE, D> : &k_batch_tile<S, FIELDS_NONE, false>)
                 : fields == FIELDS_ALL ? (d ? &k_batch_tile<S, FIELDS_ALL, D> : &k_batch_tile<S, FIELDS_ALL, false>)
                                        : (d ? &k_batch_tile<S, FIELDS_SOME, D> : &k_batch_tile<S, FIELDS_SOME, false>);
    hipLaunchKernelGGL(k, dim3(nitems), dim3(threads), 0, st, probs, items, parity, ns);
    return hipGetLastError();
}

hipError_t launch_batch_tile(int storage, const BatchProblem *probs, const int2 *items, int nitems, int fields,
                             long long nodes, int threads, int parity, int ns, hipStream_t st)
{
    switch (storage) {
    case 0: return batch_tile_t<double>(probs, items, nitems, fields, nodes, threads, parity, ns, st);
    case 1: return batch_tile_t<float>(probs, items, nitems, fields, nodes, threads, parity, ns, st);
    case 2: return batch_tile_t<__half>(probs, items, nitems, fields, nodes, threads, parity, ns, st);
    default: return hipErrorInvalidValue;
    }
}

// Tiles and steps per launch for the grids of one launch (n = 1: one problem; else a batch,
// whose problems share the steps per launch and the largest tile).
//
// Grids of at most TILE_NT nodes are one block each, which needs no overlap and takes any
// number of steps per launch.  Otherwise the tiles and steps of least estimated time per
// step are taken.  Per launch the estimate adds, in units of a round's fixed cost (launch,
// first loads, last stores: 4-6 us): one for each round of blocks on the 256 CUs; 0.05 for
// every step of a round (its chain of dependent instructions and two barriers); 0.12 for
// every node update that a SIMD issues for a wavefront.  Over 875 measured combinations on
// nine grids from 48 x 90 to 1300 x 1201 nodes the choice costs 3 % (FP64, FP16) and 5 % (FP32)
// more on average than the best one.
// It knows nothing of the memory system, which decides once the blocks come in rounds: regions of
// 32 columns read whole lines, and more steps per launch read less.  From TILE_WIDE[0] nodes on
// (grids several tiles across) it chooses between two such tiles, from TILE_WIDE[1] nodes on the
// better one is fixed per type.  us per step with the estimate's choice of all shapes and with
// these: FP32 380^2 6.4 and 4.4, 600^2 15.2 and 9.8, 1200^2 41.6 and 30.2, 1500^2 64 and 46.8 (the
// two-step pass 51.5); FP64 850^2 36.7 and 26.8; FP16 1300^2 35.8 and 32.2; of (28, 12) in 3 and (26, 10) in 4
// steps, FP32 1000^2 23.1 and 21.4, FP64 700^2 21.2 and 23.3, 1400^2 68.3 and 63.1, FP16 1000^2 20.2
// and 23.2.
//
// A narrow grid (fewer than TILE_ACROSS columns or tile_rows rows) is one or two tiles across and
// takes any shape; a batch does where such problems hold more than half of its nodes.  With the
// estimate's choice, us per step, and the wide tiles: 20,000 x 40 FP64 52.8 and 36.7, FP32 36.4 and
// 20.0, 123,076 x 26 FP32 99 and 75; but 12,121 x 33 FP64 20.1 and 22.7, 20,000 x 20 FP16 8.2 and 11.0, 7,500 x 20
// FP32 4.3 and 5.3; 64 cavities of 200^2 and one of 40^2, FP64 162 and 110, FP32 104 and 64 (the passes 117 and 73).
//
// Larger grids take the two-step pass (FP16: single steps), which is bound by HBM and recomputes less
// (TILE_NODES).  us per step here and there: FP32 1800 x 1900 66 and 67, 2500^2 120 and
// 113; FP64 1300^2 53 and 65, 1700^2 91 and 98, 2400^2 177-184 and 182, 3000^2 275 and 276; FP16 1500^2 41
// and 44, 2000^2 75 and 71.  With a porosity field, whose coefficients a tile forms once per launch,
// FP32 2000 x 2100 90 and 102, 3500^2 259 and 264; FP64 2000^2 135 and 153, 3500^2 399 and 419; FP16 1800 x 1900
// 71 and 77, 2200^2 97 and 94.
// Between walls few rows apart a third of the tiles and more hold wall nodes, whose chain is the
// longer one: there the limit is TILE_FLAT nodes, more in one or two rows of tiles, or TILE_PER_ROW per
// row.  21,276 x 47 FP64 44 and 51, 34,042 x 47 71 and 70, with a field 90 and 78, 26,666 x 60 69 and 67, 88 and 77,
// 8,000 x 200 57 and 63, 66 and 73, 16,000 x 200 113 and 111, 135 and 126, 15,000 x 400 189 and 187, 219 and 212,
// 61,538 x 26 66 and 77, 96,969 x 33 143 and 136, 333,333 x 12 108 and 211, 200,000 x 4 with a field 0.94 times;
// FP16 26,666 x 60 33.5 and 31.7, 8,000 x 200 30.6 and 31.8, 16,000 x 200 60 and 50; FP32 with a field
// 60,000 x 200 279 and 264.  FP64 grids of 48 to 63 columns, of which two tiles in three hold wall nodes and
// which fill the one wavefront of a pass: 62 x 25,806 80 and 81, with a field 96 and 93.
// Batches: FP64 cavities of 180-300 nodes a side, 3.7 M in all, 150 and 156, 8.6 M 354 and 346; FP32 of 200^2
// 4 M 112 and 123, of 500^2 3.75 M 103 and 102, of 1000^2 5 M 104 and 99; FP16 10.6 M 268 and 270, two of 1300^2 64
// and 64.
constexpr int TILE_MAX_STEPS = 8, TILE_ALL_STEPS = 1024;
constexpr long long TILE_WIDE[2] = {120000, 350000};
constexpr int TILE_ACROSS = 48;
constexpr long long TILE_NODES[3] = {5000000, 3500000, 2300000};
constexpr long long TILE_NODES_FIELD[3] = {12500000, 12500000, 4200000};
constexpr long long TILE_FLAT[3] = {1200000, 6000000, 1100000};
constexpr long long TILE_FLAT_FIELD[3] = {1200000, 6000000, 1700000};
constexpr int TILE_PER_ROW[3] = {8000, 6000, 8000};
constexpr long long TILE_NODES_BATCH[2] = {4000000, 6000000};   // FP16: the mean grid at most TILE_MEAN
constexpr long long TILE_MEAN = 1700000;
constexpr long long TILE_LARGE = 150000, TILE_NODES_LARGE = 3500000;   // FP32 batches of grids of TILE_LARGE on average

// What the plan looks at in the grids of a launch.
struct TileSet {
    int storage, n;
    long long nodes;
    bool field;                  // all with a porosity field
    bool narrow, thin;           // the narrow grids, those of fewer than TILE_ACROSS columns, hold most of the nodes
    int nx, ny;                  // n = 1
    bool px, py;
    long long flat;              // limit of the nodes between walls few rows apart
};

// Rows below which a grid is narrow, in a launch of `nodes` nodes.
static int tile_rows(int storage, long long nodes)
{
    return nodes < TILE_WIDE[1] ? TILE_ACROSS : (storage == 1 && nodes >= TILE_FLAT[0] ? 18 : 36);
}

static long long tile_flat_limit(int storage, bool field, int ny)
{
    const long long flat = (field ? TILE_FLAT_FIELD : TILE_FLAT)[storage];
    if (ny < 6 && storage == 0) return 750000;
    if (ny < 20) return INT64_MAX;
    return std::max(ny < 36 ? flat * 4 / 3 : flat, (long long)TILE_PER_ROW[storage] * ny);
}

static long long tile_nodes_limit(const TileSet &t)
{
    if (t.n > 1) {
        if (t.storage == 2) return std::min(t.flat, t.n * TILE_MEAN);
        const bool large = t.storage == 1 && !t.field && t.nodes >= t.n * TILE_LARGE;
        return std::min(t.flat, large ? TILE_NODES_LARGE : TILE_NODES_BATCH[t.storage]);
    }
    const long long most = (t.field ? TILE_NODES_FIELD : TILE_NODES)[t.storage];
    if (t.storage == 0 && !t.px && t.nx >= TILE_ACROSS && t.nx < 64) return std::min(most, TILE_FLAT[0]);
    return std::min(most, t.flat);
}

// Fewest steps of a launch.  A launch costs about the same for any number of steps once a grid fills
// the chip (FP32 1800 x 1900 245 us for one step, 264 for four): the steps that are left over from
// full launches, and short calls, go to the passes where those are faster: from TILE_STEPS1, 2 and 3
// nodes on for one, two and three steps.  us per step here and there: one, FP64 420 x 427 19.2 and
// 21.0, 500 x 507 27.1 and 24.2, FP32 500 x 507 15.2 and 17.1, 640 x 647 28.6 and 22.3, FP16 720 x 727 18.9 and
// 21.0, 850 x 857 28.9 and 23.6; two, FP64 850 x 857 40 and 44, 1150 x 1157 70 and 61, FP32 950 x 957 34.5 and
// 39.1, 1150 x 1157 49.5 and 39.0, FP16 950 x 957 24.0 and 26.4, 1150 x 1157 33.7 and 30.6; three, FP32 1550 x 1557
// 62 and 63, 1750 x 1757 81 and 75, with a field 1650 x 1657 75 and 80, 1850 x 1857 100 and 95 (FP64: never,
// 2200^2 191 and 195).
// Walls few nodes apart make tiles slower as above (one step, FP64 124 x 1209 17.2 and 13.8, FP32 14,705 x 17
// 19.0 and 15.5; two, FP32 30,303 x 33 40.8 and 34.6; three 60,606 x 33 64 and 57, FP64 with a field 27,777 x 36
// 69 and 59): such grids count TILE_NEAR_BY times.  A pass's wavefronts take 62 columns (FP16: 64) and leave
// lanes idle beside a grid that is not a multiple (one step, FP64 with a field 64 x 3906 32 and 42, FP32
// 64 x 9375 51 and 42; two, FP32 64 x 37,500 99 and 126, 80 x 30,000 0.9 times): the square of the share of the
// lanes in use enters.  Up to TILE_THIN columns tiles are faster in any case (one step, 32 x 100,000
// FP64 309 and 388), below TILE_ACROSS for two steps and more (40 x 60,000 158 and 186), in FP16 below
// TILE_NEAR (80 x 30,000 with a field 77 and 144).
// Batches: one step, FP64 16 of 200^2 0.99 times, FP32 10 of 200^2 1.02 and 16 0.84, FP16 10 of 200^2 1.27 and
// 16 0.92; two, FP64 25 of 200^2 1.04 and 40 0.86, FP32 1.05 and 0.93, FP16 six of 500^2 1.11 and 12
// 0.99; three, FP32 ten of 500^2 1.03 and 12 0.99; 200 of 47 x 400, FP32, one step 276 and 336 us.
constexpr long long TILE_STEPS1[3] = {180000, 270000, 450000}, TILE_STEPS2[3] = {800000, 1000000, 850000};
constexpr long long TILE_STEPS3[2] = {2500000, 3000000};                        // FP32; with a field
constexpr long long TILE_STEPS3_FLAT[3] = {900000, 1800000, 1500000};           // FP64 with a field, FP32, FP16 one or two tiles high
constexpr int TILE_THIN = 32, TILE_NEAR = 150;
constexpr double TILE_NEAR_BY[2][3] = {{2.0, 1.7, 1.6}, {1.2, 1.15, 1.5}};      // for one and for two steps
constexpr long long TILE_STEPS1_BATCH[3] = {550000, 430000, 600000}, TILE_STEPS2_BATCH[3] = {1050000, 1200000, 2500000};
constexpr long long TILE_STEPS3_BATCH = 2800000;                                // FP32, grids of TILE_LARGE on average
constexpr long long TILE_SMALL = 100000;                                        // FP16: grids below on average, any two

// Launches that store every step (the adjoint's forward states) write tiles of 24-28 columns, parts of
// cache lines, once per step.  us per reverse step by tiles and by single steps: FP64 576^2 75.6 and 77.0,
// 768^2 125 and 122, 1024^2 212 and 188; FP32 450^2 38.0 and 40.6, 576^2 65.0 and 61.9, 1024^2 181 and 144, 1536^2
// 400 and 314; FP16 768^2 91 and 94, 1024^2 143 and 139.
constexpr long long TILE_EVERY[3] = {500000, 280000, 800000};

static int tile_least_batch(const TileSet &t)
{
    if ((t.thin && t.storage != 0) || t.nodes < TILE_STEPS1_BATCH[t.storage]) return 1;
    if (t.nodes < TILE_STEPS2_BATCH[t.storage] || (t.storage == 2 && t.nodes < t.n * TILE_SMALL)) return 2;
    return t.storage == 1 && t.nodes >= std::max(TILE_STEPS3_BATCH, t.n * TILE_LARGE) ? 4 : 3;
}

static int tile_least(const TileSet &t)
{
    if (t.n > 1) return tile_least_batch(t);
    if (t.nx <= TILE_THIN) return 1;
    const int s = t.storage, cols = s == 2 ? 64 : 62, chunks = (t.nx + cols - 1) / cols;
    const double used = (double)t.nx / ((double)chunks * cols), nodes = (double)t.nodes * used * used;
    const bool flat = !t.py && t.ny < TILE_NEAR, tall = !t.px && t.nx < TILE_NEAR;
    const bool near = tall || (flat && (s == 0 || t.ny > 16));  // FP32 and FP16: not if one tile holds both walls
    if (nodes * (near ? TILE_NEAR_BY[0][s] : 1.0) < (double)TILE_STEPS1[s]) return 1;
    if (t.nx < TILE_ACROSS || (s == 2 && tall)) return 2;
    if (nodes * (near ? TILE_NEAR_BY[1][s] : 1.0) < (double)TILE_STEPS2[s]) return 2;
    const bool by_flat = flat && (s == 0 ? t.field : (s == 1 ? t.ny > 16 : t.narrow));
    if (by_flat && t.nodes >= TILE_STEPS3_FLAT[s]) return 4;
    return s == 1 && t.ny > 16 && nodes >= (double)TILE_STEPS3[t.field] ? 4 : 3;
}

struct TileShape { int tw, th, ns0, ns1; };       // tile and the range of steps per launch
struct TileShapes { const TileShape *first; int n; };

// The shapes that tile_plan chooses from.
static TileShapes tile_shapes(const TileSet &t)
{
    constexpr int M = TILE_MAX_STEPS;
    static constexpr TileShape all[] = {{8, 8, 1, M}, {12, 8, 1, M}, {16, 8, 1, M}, {32, 8, 1, M}, {12, 12, 1, M}, {16, 12, 1, M},
                                        {16, 16, 1, M}, {20, 20, 1, M}, {28, 12, 1, M}, {26, 10, 1, M}, {30, 14, 1, M}};
    static constexpr TileShape large[] = {{28, 12, 3, 3}, {26, 10, 4, 4}};
    if (!t.narrow && t.nodes >= TILE_WIDE[1]) return {large + (t.storage == 1 || tile_dense(t.storage, t.nodes)), 1};
    if (!t.narrow && t.nodes >= TILE_WIDE[0]) return {large, 2};
    return {all, (int)(sizeof(all) / sizeof(all[0]))};
}

TileSteps tile_plan(int storage, const KParams *P, int n, TileGrid *grids)
{
    TileSet t = {};
    t.storage = storage;
    t.n = n;
    t.field = true;
    t.nx = P[0].nx; t.ny = P[0].ny; t.px = P[0].px; t.py = P[0].py;
    t.flat = INT64_MAX;
    bool one_block = true;
    for (int k = 0; k < n; ++k) {
        t.nodes += (long long)P[k].nx * P[k].ny;
        t.field = t.field && P[k].field;
    }
    long long narrow = 0, thin = 0;
    const int rows = tile_rows(storage, t.nodes);
    for (int k = 0; k < n; ++k) {
        const long long nk = (long long)P[k].nx * P[k].ny;
        one_block = one_block && nk <= TILE_NT;
        if (P[k].nx < TILE_ACROSS) thin += nk;
        if (P[k].nx < TILE_ACROSS || P[k].ny < rows) narrow += nk;
        // a batch of grids that are not flat has the same share of wall nodes in its passes
        if (!P[k].py && (n == 1 || P[k].nx >= 8 * (long long)P[k].ny))
            t.flat = std::min(t.flat, tile_flat_limit(storage, t.field, P[k].ny));
    }
    t.narrow = 2 * narrow > t.nodes;
    t.thin = 2 * thin > t.nodes;
    if (t.nodes > tile_nodes_limit(t)) return {0, 0, false};
    if (one_block) {
        for (int k = 0; k < n; ++k) grids[k] = tile_grid(P[k], P[k].nx, P[k].ny);
        // one step of more than 256 nodes between x walls: 22 x 22 FP64 7.7 us here and 6.6, FP32 6.6 and
        // 5.5 (periodic in x 7.4 and 9.5; 16 x 16 6.9 and 6.7)
        return {TILE_ALL_STEPS, n == 1 && storage != 2 && !t.px && t.nodes > 256 ? 2 : 1, true};
    }
    const int resident = storage == 0 ? 8 : 16;   // wavefronts of this kernel that a CU's registers hold
    const double cus = 256.0;
    TileShape shape = {};
    int best = 0;
    double cost = 0.0;
    const TileShapes shapes = tile_shapes(t);
    for (int i = 0; i < shapes.n; ++i) {
        const TileShape &sh = shapes.first[i];
        for (int ns = sh.ns0; ns <= sh.ns1; ++ns) {
            double blocks = 0.0, updates = 0.0;   // over all grids: blocks; node updates of a wavefront
            int waves = 0;                        // of the largest block
            for (int k = 0; k < n && waves >= 0; ++k) {
                const TileGrid g = tile_grid(P[k], sh.tw, sh.th);
                int w, h;
                tile_extent(g, ns, w, h);
                if ((g.nbx > 1 && g.tw < 4) || (g.nby > 1 && g.th < 4) || w * h > TILE_NT) {
                    waves = -1;
                    break;
                }
                const double nb = (double)g.nbx * g.nby;
                int u = 0;
                for (int s = 0; s < ns; ++s) u += (w * (g.nby > 1 ? h - 2 * s : h) + 63) / 64;
                blocks += nb;
                updates += nb * u;
                waves = std::max(waves, (w * h + 63) / 64);
            }
            if (waves < 0) break;
            const double percu = std::max(1, resident / waves);
            const double rounds = std::ceil(blocks / (cus * percu));
            const double simd = std::ceil(blocks / cus) * (updates / blocks) / 4.0;
            const double c = (rounds + 0.05 * rounds * ns + 0.12 * simd) / ns;
            if (best == 0 || c < cost) {
                cost = c;
                best = ns;
                shape = sh;
            }
        }
    }
    for (int k = 0; k < n && best; ++k) grids[k] = tile_grid(P[k], shape.tw, shape.th);
    return {best, std::min(best, tile_least(t)), t.nodes < TILE_EVERY[storage]};
}

int tile_threads(const TileGrid &g, int ns)
{
    int w, h;
    tile_extent(g, ns, w, h);
    return (w * h + 63) / 64 * 64;
}

}  // namespace lbm
