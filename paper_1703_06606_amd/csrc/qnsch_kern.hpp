// qnsch_kern.hpp -- work-list kernels of the FP64 multigrid step.
//
// Every kernel takes a work list: up to MAXITEMS items, each naming one level
// of one simulation (a device descriptor) and the range of workgroups that
// work on it.  A launch therefore applies the same operation (a colour
// half-sweep, a restriction, ...) to many simulations at once, at whatever
// level each of them is; a single simulation is a list of one item.  The
// work of a workgroup depends only on its item, so a simulation's results do
// not depend on what else shares the launch.
#pragma once
#include <type_traits>

#include "qnsch_dev.hpp"
#include "qnsch_lin.hpp"

namespace qn {

#define BLK 256
#define NRED 16 // reduction slots
// Tile of cells per workgroup (one lane pair per cell of a colour).  16 x 16
// cells and 256 lanes: small levels spread over more CUs, and two or three
// workgroups share a CU on large ones (measured against 32 x 16 and 32 x 8).
#ifndef QN_TX
#define QN_TX 16
#endif
#ifndef QN_TY
#define QN_TY 16
#endif
#define TX QN_TX
#define TY QN_TY
#define TBLK (TX * TY)
#define HS_ATTR __launch_bounds__(TBLK)
#define TILE_S (TX + 4)
#define TILE_DOUBLES (T_ES * TILE_S * (TY + 3))
#define TILE_LDS __shared__ __attribute__((aligned(16)))
#define NXCD 8
#define MAXITEMS 64
static_assert(TILE_DOUBLES * 8 + 16 * NRED * 8 <= 65536, "tile exceeds 64 KiB of LDS");

// one level of one simulation, in device memory; the levels of a simulation
// follow each other, so that the next coarser one's is the next descriptor
struct Desc {
    Phys P;
    Kon<double> K;
    double *c, *mu, *p, *ub[2], *vb[2], *cn, *un, *vn; // level arrays (u/v ping-pong)
    double *fc, *fmu, *fp, *fu, *fv;                    // FAS right-hand side (NULL on the finest level)
    double *c0, *mu0, *p0, *u0, *v0;                    // restricted iterate (coarse levels)
    int m1, m2, pitch, bcx, bcy;
    int depth;                                          // levels from this one to the coarsest, both included
    double h, inv_h;
    double *partials;                                   // per-simulation reduction partials (finest level)
    double *red;                                        // reduced values (device)
    double *red_host;                                   // reduced values (pinned host)
    double *mus, *ps;                                   // mubar, pbar of time n (finest level)
    double *c2, *mu2, *p2;                              // second set of cell unknowns (fused sweeps; else NULL)
    double *rout;                                       // residual fields (finest level, optional)
    // acceleration history (finest level): a ring of am slots, each holding
    // a cycle result (aw, pbar before its mean removal) and its residual (ar)
    // as 5 fields of pitch*m2, and the pbar mean removed from it (amean)
    double *aw, *ar, *amean;
    int am;
    // mixed precision: the FP32 correction hierarchy (NULL in FP64 mode; on
    // coarse levels the FP64 arrays above are NULL instead)
    PhysF Pf;
    Kon<float> Kf;
    float *xc, *xmu, *xu, *xv;                          // linearisation point
    float *dc, *dmu, *dp, *dub[2], *dvb[2];             // correction (u/v ping-pong)
    float *rc, *rmu, *rp, *ru, *rv;                     // right-hand side
    float *dc2, *dmu2, *dp2;                            // second set of cell corrections (fused sweeps)
    float *cnf, *unf, *vnf;                             // time-n data
};

// (The small entries are 32-bit: a kernel reads them with scalar loads,
// which have no 16-bit form; a 16-bit entry cost a vector load and its
// memory latency at the start of every kernel.)
struct Items {
    int n;
    int start[MAXITEMS + 1];  // first workgroup of each item; start[n] = total
    const Desc *d[MAXITEMS];  // the level worked on
    int par[MAXITEMS];        // current u/v buffer of that level
    int cpar[MAXITEMS];       // current u/v buffer of the next coarser level
    int tx[MAXITEMS];         // tiles per row (tile kernels); partial count (k_finalize)
    int acc[MAXITEMS];        // acceleration ring slot s | (earlier results used) << 4; -1 none
};
// A list of one item (a simulation run on its own), as five kernel arguments of
// 28 bytes in all.  They arrive in scalar registers with the wave (kernel
// argument preloading), so that a kernel's first memory access is the level
// descriptor's: read from memory, as the many-item list's 1.8 KB are, the
// arguments cost every kernel a round trip of ~0.5 us before it, and a
// dependent launch another 1.5 us for 1.4 KB of them.
// w: u/v buffer of the level, of the next coarser one << 1, (acceleration
// slot and earlier results, or -1) + 1 << 2; cnt: tiles per row, or partials.
// base, geom: where the level's arrays are (Lay), for the smoothing and residual
// kernels, whose first reads are its fields: these start with the wave then, and
// the descriptor's constants come behind them, instead of behind some eight
// scalar reads that wait for each other (one fused sweep of 256 tiles 10.2 us
// against 9.3, two of 32 tiles 13.5 against 13.1, the half-sweep of 1024 tiles
// 13.1 against 12.5).  NULL: the arrays are the descriptor's.  (The restriction
// and the bottom levels, which read several descriptors in any case, and FP32
// gained nothing: 5.7 against 6.0 us, 53.8 against 54.7, two sweeps 10.3 against
// 10.4.)
struct Item1 {
    const Desc *d;
    int w, cnt;
    const char *base;
    unsigned geom;
};

__device__ __forceinline__ int find_item(const Items &it)
{
    int k = 0;
    while (k + 1 < it.n && (int)blockIdx.x >= it.start[k + 1]) k++;
    return k;
}
__device__ __forceinline__ int find_item(const Item1 &) { return 0; }
__device__ __forceinline__ const Desc &it_desc(const Items &it, int k) { return *it.d[k]; }
__device__ __forceinline__ const Desc &it_desc(const Item1 &it, int) { return *it.d; }
__device__ __forceinline__ int it_par(const Items &it, int k) { return it.par[k]; }
__device__ __forceinline__ int it_par(const Item1 &it, int) { return it.w & 1; }
__device__ __forceinline__ int it_cpar(const Items &it, int k) { return it.cpar[k]; }
__device__ __forceinline__ int it_cpar(const Item1 &it, int) { return (it.w >> 1) & 1; }
__device__ __forceinline__ int it_cnt(const Items &it, int k) { return it.tx[k]; }
__device__ __forceinline__ int it_cnt(const Item1 &it, int) { return it.cnt; }
__device__ __forceinline__ int it_acc(const Items &it, int k) { return it.acc[k]; }
__device__ __forceinline__ int it_acc(const Item1 &it, int) { return (it.w >> 2) - 1; }
__device__ __forceinline__ int it_start(const Items &it, int k) { return it.start[k]; }
__device__ __forceinline__ int it_start(const Item1 &, int) { return 0; }

// The two kernels of an operation, NAME for a list of one item and NAME_n for
// many, from its body NAME_body(list, ...).  PARAMS, ARGS: the further
// parameters, in parentheses.  QN_KERNEL_PJ: a body with the template
// parameter PJ (projection scheme; not served, so no NAME_n of it).  QN_KERNEL1,
// QN_KERNEL1_PJ: without NAME_n (operations that the server does not use).
#define QN_MORE(...) , ##__VA_ARGS__
#define QN_KERNEL1(NAME, ATTR, PARAMS, ARGS)                                                       \
    __global__ ATTR void NAME(const Desc *__restrict__ d, int w, int cnt, const char *base, unsigned geom QN_MORE PARAMS) \
    {                                                                                              \
        NAME##_body(Item1{ d, w, cnt, base, geom } QN_MORE ARGS);                                  \
    }
#define QN_KERNEL(NAME, ATTR, PARAMS, ARGS)                                                        \
    QN_KERNEL1(NAME, ATTR, PARAMS, ARGS)                                                           \
    __global__ ATTR void NAME##_n(Items it QN_MORE PARAMS) { NAME##_body(it QN_MORE ARGS); }
#define QN_KERNEL1_PJ(NAME, ATTR, PARAMS, ARGS)                                                    \
    template <bool PJ> __global__ ATTR void NAME(const Desc *__restrict__ d, int w, int cnt, const char *base, unsigned geom QN_MORE PARAMS) \
    {                                                                                              \
        NAME##_body<PJ>(Item1{ d, w, cnt, base, geom } QN_MORE ARGS);                              \
    }
#define QN_KERNEL_PJ(NAME, ATTR, PARAMS, ARGS)                                                     \
    QN_KERNEL1_PJ(NAME, ATTR, PARAMS, ARGS)                                                        \
    __global__ ATTR void NAME##_n(Items it QN_MORE PARAMS) { NAME##_body<false>(it QN_MORE ARGS); }

__device__ __forceinline__ View view_of(const Desc &d, int par)
{
    View V;
    V.c = d.c; V.mu = d.mu; V.p = d.p;
    V.u = d.ub[par]; V.v = d.vb[par];
    V.cn = d.cn; V.un = d.un; V.vn = d.vn;
    V.m1 = d.m1; V.m2 = d.m2; V.pitch = d.pitch;
    V.bcx = d.bcx; V.bcy = d.bcy;
    V.inv_h = d.inv_h;
    return V;
}
// The FP64 arrays of a level lie one after the other, ARR_* arrays of the same
// size (rounded up to 256 bytes), and levels follow each other.  geom: cells,
// boundary kinds, whether there is a second set of cell unknowns, whether the
// level is the finest (which has no right-hand sides and restricted iterate).
enum { ARR_C, ARR_MU, ARR_P, ARR_U0, ARR_V0, ARR_U1, ARR_V1, ARR_CN, ARR_UN, ARR_VN, ARR_C2, ARR_RHS = ARR_C2, ARR_W0 = ARR_RHS + 5,
       ARR_END = ARR_W0 + 5 };
#define GEOM_MAX 0x3fff
static __host__ __device__ __forceinline__ size_t arr_bytes(int m1, int m2) { return ((size_t)m1 * m2 * sizeof(double) + 255) & ~(size_t)255; }
struct Lay {
    const char *base;
    int m1, m2, bcx, bcy, two, fine;
    __device__ __forceinline__ double *arr(int k) const { return (double *)(base + k * arr_bytes(m1, m2)); }
    __device__ __forceinline__ double *set2(int k) const { return arr(ARR_C2 + k); }
    __device__ __forceinline__ double *rhs(int k) const { return arr(ARR_RHS + 3 * two + k); }
    __device__ __forceinline__ double *w0(int k) const { return arr(ARR_W0 + 3 * two + k); }
    __device__ __forceinline__ double *u(int par) const { return arr(par ? ARR_U1 : ARR_U0); }
    __device__ __forceinline__ double *v(int par) const { return arr(par ? ARR_V1 : ARR_V0); }
    __device__ __forceinline__ Lay next() const
    {
        Lay n = *this;
        n.base = (const char *)arr((fine ? (int)ARR_RHS : (int)ARR_END) + 3 * two);
        n.m1 >>= 1;
        n.m2 >>= 1;
        n.fine = 0;
        return n;
    }
};
__device__ __forceinline__ Lay lay_of(const Item1 &it)
{
    const unsigned g = it.geom;
    return { it.base, (int)(g & GEOM_MAX), (int)(g >> 14 & GEOM_MAX), (int)(g >> 28 & 1), (int)(g >> 29 & 1), (int)(g >> 30 & 1),
             (int)(g >> 31) };
}
__device__ __forceinline__ View view_of(const Items &, const Desc &d, int par) { return view_of(d, par); }
__device__ __forceinline__ View view_of(const Lay &L, int par)
{
    View V;
    V.c = L.arr(ARR_C); V.mu = L.arr(ARR_MU); V.p = L.arr(ARR_P);
    V.u = L.u(par); V.v = L.v(par);
    V.cn = L.arr(ARR_CN); V.un = L.arr(ARR_UN); V.vn = L.arr(ARR_VN);
    V.m1 = L.m1; V.m2 = L.m2; V.pitch = L.m1;
    V.bcx = L.bcx; V.bcy = L.bcy;
    V.inv_h = 0.0; // (not a tile kernel's)
    return V;
}
__device__ __forceinline__ View view_of(const Item1 &it, const Desc &d, int par)
{
    return it.base ? view_of(lay_of(it), par) : view_of(d, par);
}
// the level's constants: of one item the descriptor, read where they are used,
// behind the first loads; of a list a copy, read before a kernel's first store
// (its descriptors are not known to be apart from the stores: read later, their
// fields would be vector loads)
struct Consts {
    Phys P;
    Kon<double> K;
};
__device__ __forceinline__ Consts consts_of(const Items &, const Desc &d) { return { d.P, d.K }; }
__device__ __forceinline__ const Desc &consts_of(const Item1 &, const Desc &d) { return d; }
// what a smoothing kernel reads and writes of a level: its right-hand sides
// (none on a finest level), the other u/v buffer, the second set of cells
struct LevOut {
    Rhs F;
    double *un, *vn, *c2, *mu2, *p2;
};
__device__ __forceinline__ LevOut out_of(const Desc &d, int par)
{
    return { { d.fc, d.fmu, d.fp, d.fu, d.fv }, d.ub[par ^ 1], d.vb[par ^ 1], d.c2, d.mu2, d.p2 };
}
__device__ __forceinline__ LevOut out_of(const Items &, const Desc &d, int par) { return out_of(d, par); }
__device__ __forceinline__ LevOut out_of(const Item1 &it, const Desc &d, int par)
{
    if (!it.base) return out_of(d, par);
    const Lay L = lay_of(it);
    LevOut o = { {}, L.u(par ^ 1), L.v(par ^ 1), L.set2(0), L.set2(1), L.set2(2) };
    if (!L.fine) o.F = { L.rhs(0), L.rhs(1), L.rhs(2), L.rhs(3), L.rhs(4) };
    return o;
}
__device__ __forceinline__ int it_m2(const Items &, const Desc &d) { return d.m2; }
__device__ __forceinline__ int it_m2(const Item1 &it, const Desc &d) { return it.base ? (int)(it.geom >> 14 & GEOM_MAX) : d.m2; }
__device__ __forceinline__ Rhs rhs_of(const Desc &d)
{
    const Rhs F = { d.fc, d.fmu, d.fp, d.fu, d.fv };
    return F;
}

// Workgroups are dispatched round-robin over the XCDs, each with its own L2.
// Items of many tiles start at multiples of NXCD and their tiles are renumbered
// so that an XCD gets a contiguous band of tiles: neighbouring tiles, which
// read each other's halos, share one L2.
// (TS: the side of a square tile; it_cnt holds the tiles per row)
template <int TS, typename IT> __device__ __forceinline__ int item_tile_at(const IT &it, int k, const Desc &d, int &i0, int &j0)
{
    const int tx = it_cnt(it, k), ty = (it_m2(it, d) + TS - 1) / TS;
    const int n = tx * ty, lin = (int)blockIdx.x - it_start(it, k);
    const int t = (n % NXCD == 0) ? (lin % NXCD) * (n / NXCD) + lin / NXCD : lin;
    i0 = (t % tx) * TS;
    j0 = (t / tx) * TS;
    return lin < n;
}
// places per slot of a simulation's partials: as many as its finest level has
// tiles (no fewer than blocks of BLK cells)
__device__ __forceinline__ int part_stride(const Desc &d) { return ((d.m1 + TX - 1) / TX) * ((d.m2 + TY - 1) / TY); }

// (W: the elements that the tile's cells read, -1 .. TX+1 along an axis for a
// box, whose high face is an unknown, -1 .. TX for a residual)
template <typename TT, int W = TX + 3, int S = TILE_S, typename R, typename IT>
__device__ __forceinline__ TT item_tile(R *sm, const IT &it, int k, const Desc &d)
{
    static_assert(TX == TY, "square tiles");
    TT T;
    T.s = sm;
    item_tile_at<TX>(it, k, d, T.i0, T.j0);
    T.W = W;
    T.H = W;
    T.S = S;
    return T;
}
template <typename IT> __device__ __forceinline__ bool tile_valid(const IT &it, int k, const Desc &d)
{
    return (int)blockIdx.x - it_start(it, k) < it_cnt(it, k) * ((it_m2(it, d) + TY - 1) / TY);
}

// --------------------------------------------------------------------------
// one colour half-sweep (sec. 7.1) on a tile: a lane pair per cell of the
// colour.  The u/v snapshot is buffer par, the new faces go to buffer par^1.
template <bool PJ, bool RHS = true, typename IT> __device__ __forceinline__ void k_halfsweep_body(const IT &it, int colour, double omega)
{
    TILE_LDS double sm[TILE_DOUBLES];
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    if (!tile_valid(it, k, d)) return;
    const int par = it_par(it, k);
    const View L = view_of(it, d, par);
    const Tile T = item_tile<Tile>(sm, it, k, d);
    const LevOut o = out_of(it, d, par);
    const auto &dc = consts_of(it, d);
    tile_load<2, TBLK>(dc, L, T);
    const Phys P = dc.P;
    const Kon<double> K = dc.K;
    const Rhs F = RHS ? o.F : Rhs();
    double *const un = o.un, *const vn = o.vn;
    __syncthreads();
    const int pr = threadIdx.x >> 1, hlf = threadIdx.x & 1;
    const int lj = pr / (TX / 2), kk = pr - lj * (TX / 2);
    const int j = T.j0 + lj;
    const int i = T.i0 + 2 * kk + ((j + colour) & 1);
    if (i < L.m1 && j < L.m2) relax_cell<PJ, 0, 1, false>(P, K, L, T, F, un, vn, i, j, i, j, hlf, omega, 1.0);
}
QN_KERNEL_PJ(k_halfsweep, HS_ATTR, (int colour, double omega), (colour, omega))
// the same for launches whose items are all finest levels, which have no
// right-hand sides (512 x 2048: 37.5 us with them, 36.2 without), under its own
// name, so that profiles tell the finest level apart.  What bounds it there:
// neither memory (105 MB, 2.9 TB/s) nor the vector units (19 us of issue), but
// three workgroups per CU, by registers and LDS, that load, relax and store in
// turn.  A lane per cell on tiles of 32 x 16 (35 % fewer instructions, two
// workgroups per CU) took 37.3 us, workgroups that stay and prefetch their next
// tile 48, four waves per SIMD at the price of spills 48.
template <bool PJ, typename IT> __device__ __forceinline__ void k_halfsweep_fine_body(const IT &it, int colour, double omega)
{
    k_halfsweep_body<PJ, false>(it, colour, omega);
}
QN_KERNEL_PJ(k_halfsweep_fine, HS_ATTR, (int colour, double omega), (colour, omega))

// --------------------------------------------------------------------------
// temporal blocking: NS sweeps (each a red, then a black half-sweep of sec. 7.1,
// the same arithmetic as two k_halfsweep launches) in one launch.  A workgroup
// loads its tile of TS x TS cells with everything that its last half-sweep
// depends on, and each half-sweep relaxes a region two cells narrower on every
// side than the one before, in LDS (neighbouring workgroups compute the
// overlap again); the last one covers the tile.  Workgroups still read their
// neighbours' cells as halo while others write, so the cell unknowns go from
// one set to the other (dir 0: c, mu, p to c2, mu2, p2; dir 1 back) and the
// faces from buffer par to par ^ 1.
// Threads: the tile's 23 x 23 elements load in one round (512 threads take a
// second one for 17 elements: one sweep of 128 x 256 cells 10.3 us against 9.7,
// two of 64 x 128 13.8 against 13.7, FP32 11.0 against 10.4).  Nine waves may have
// 168 registers each: the FP64 kernels then spill 12 (one sweep) and 20 bytes
// (two) per lane, none with 512 threads, which the times above include.  The
// projection scheme's 177 registers do not fit (13.7 against 15.6 us).
#define FUSED_BLK(PJ) ((PJ) ? 2 * TBLK : 2 * TBLK + 64)
template <int NS, int TS> struct Fused {
    static constexpr int EXT = 4 * NS - 2;         // the first region: the tile widened by EXT cells
    static constexpr int W = TS + 2 * EXT + 3;     // rows and columns loaded
    static constexpr int S = W + 1;                // row stride (even)
    static constexpr int LDS = S * W;              // elements of LDS
};

// the coarse level's arrays that the coarse-grid correction reads, and the
// fine level's boundary kinds, taken from the level descriptors once per
// workgroup (read inside the tile loader, the descriptors would be reloaded
// per element behind the tile stores)
struct PSrc {
    const double *c, *c0, *mu, *mu0, *p, *p0, *u, *u0, *v, *v0;
    int pitch, m1, m2, bcx, bcy;
};
__device__ __forceinline__ PSrc psrc_of(const Desc &d, const Desc *cp, int cpar)
{
    // the descriptor is in global memory: read through a global pointer, its
    // fields are scalar loads issued at once (a generic pointer would make
    // them vector loads)
    const __attribute__((address_space(1))) Desc &C = *(const __attribute__((address_space(1))) Desc *)cp;
    PSrc s;
    s.c = C.c; s.c0 = C.c0; s.mu = C.mu; s.mu0 = C.mu0; s.p = C.p; s.p0 = C.p0;
    s.u = C.ub[cpar]; s.u0 = C.u0; s.v = C.vb[cpar]; s.v0 = C.v0;
    s.pitch = C.pitch; s.m1 = C.m1; s.m2 = C.m2; s.bcx = d.bcx; s.bcy = d.bcy;
    return s;
}
// The coarse-grid correction P(w_H - R w_h) of the fine unknowns: a cell takes
// its coarse cell's value (piecewise constant); a face copies the coincident
// coarse face, or, between two coarse faces, averages them; a face on a wall
// is no unknown.  For one tile element it comes in two parts so that every
// load is in flight before any value is used.  prolong_load reads the coarse
// cell of the cell source (ic, jc) with its restricted iterate, and for each
// face source the coarse face it lies on and the next one along its axis (the
// periodic image, or, where there is none, the same face again: loaded, not
// used).
struct PRaw {
    double c, c0, mu, mu0, p, p0, u[4], v[4];
};
__device__ __forceinline__ PRaw prolong_load(const PSrc &C, int ic, int jc, int iu, int ju, int iv, int jv)
{
    PRaw r;
    const size_t kc = (size_t)(jc >> 1) * C.pitch + (ic >> 1);
    r.c = lda<1>(C.c, kc); r.c0 = lda<1>(C.c0, kc); r.mu = lda<1>(C.mu, kc); r.mu0 = lda<1>(C.mu0, kc);
    r.p = lda<1>(C.p, kc); r.p0 = lda<1>(C.p0, kc);
    {
        const int I = iu >> 1, J = ju >> 1;
        const size_t k0 = (size_t)J * C.pitch + I;
        const size_t k1 = I + 1 < C.m1 ? k0 + 1 : (C.bcx ? (size_t)J * C.pitch : k0);
        r.u[0] = lda<1>(C.u, k0); r.u[1] = lda<1>(C.u0, k0); r.u[2] = lda<1>(C.u, k1); r.u[3] = lda<1>(C.u0, k1);
    }
    {
        const int I = iv >> 1, J = jv >> 1;
        const size_t k0 = (size_t)J * C.pitch + I;
        const size_t k1 = J + 1 < C.m2 ? k0 + C.pitch : (C.bcy ? (size_t)I : k0);
        r.v[0] = lda<1>(C.v, k0); r.v[1] = lda<1>(C.v0, k0); r.v[2] = lda<1>(C.v, k1); r.v[3] = lda<1>(C.v0, k1);
    }
    return r;
}
// ... and the corrections: the cell unknowns, the u face (iu, ju) and the v
// face (iv, jv) (zero for a face on a wall)
__device__ __forceinline__ void prolong_apply(const PSrc &C, const PRaw &r, int iu, int iv, int jv, double &c,
                                              double &mu, double &p, double &du, double &dv)
{
    c = r.c - r.c0;
    mu = r.mu - r.mu0;
    p = r.p - r.p0;
    du = r.u[0] - r.u[1];
    if (iu & 1) {
        const double e = ((iu >> 1) + 1 < C.m1 || C.bcx) ? r.u[2] - r.u[3] : 0.0;
        du = 0.5 * (du + e);
    }
    if (!(C.bcx || iu >= 1)) du = 0.0;
    dv = r.v[0] - r.v[1];
    if (jv & 1) {
        const double e = ((jv >> 1) + 1 < C.m2 || C.bcy) ? r.v[2] - r.v[3] : 0.0;
        dv = 0.5 * (dv + e);
    }
    if (!(C.bcy || jv >= 1)) dv = 0.0;
}

__device__ __forceinline__ PSrc psrc_of(const Item1 &it, const Desc &d, int cpar)
{
    if (!it.base) return psrc_of(d, &d + 1, cpar);
    const Lay C = lay_of(it).next();
    return { C.arr(ARR_C), C.w0(0), C.arr(ARR_MU), C.w0(1), C.arr(ARR_P), C.w0(2), C.u(cpar), C.w0(3), C.v(cpar), C.w0(4),
             C.m1, C.m1, C.m2, C.bcx, C.bcy };
}

// the widened tile: every field at tile positions i0-1 .. i0+W-2 (level
// coordinates; periodic images at their unwrapped positions), the faces in both
// slots.  A periodic axis needs m >= TS + EXT + 1 so that a single wrap reaches
// every position.  With prolong set (the first sweep of a post-smoothing), each
// unknown first takes the coarse-grid correction P(w_H - R w_h) of its source
// (k_prolong's arithmetic); the sweeps write every unknown of the level, so
// the corrected values need no store of their own.
template <int NT, typename D> __device__ __forceinline__ void fused_load(const D &d, const View &L, const Tile &T, bool prolong, const PSrc &pc)
{
    const int n = T.W * T.H;
    for (int e = threadIdx.x; e < n; e += NT) {
        const int b = e / T.W, a = e - b * T.W;
        int i = T.i0 - 1 + a, j = T.j0 - 1 + b;
        if (L.bcx) i = wrapi(i, L.m1);
        if (L.bcy) j = wrapi(j, L.m2);
        const TileSrc q = tile_src(L.m1, L.m2, L.pitch, L.bcx, L.bcy, i, j);
        if (q.sc == 0) {
            tile_zero(T, b * T.S + a);
            continue;
        }
        double v[8] = { lda<1>(L.c, q.c), lda<1>(L.mu, q.c), lda<1>(L.p, q.c), lda<1>(L.u, q.u),
                        lda<1>(L.v, q.v), lda<1>(L.cn, q.c), lda<1>(L.un, q.u), lda<1>(L.vn, q.v) };
        PRaw raw = {};
        int iu = 0, iv = 0, jv = 0;
        if (prolong) {
            iu = q.u % L.pitch;
            iv = q.v % L.pitch;
            jv = q.v / L.pitch;
            raw = prolong_load(pc, q.c % L.pitch, q.c / L.pitch, iu, q.u / L.pitch, iv, jv);
        }
        // every load above is issued before anything uses a loaded value (the
        // scheduler otherwise interleaves uses with the loads, one memory
        // latency each)
        __builtin_amdgcn_sched_barrier(0);
        const Phys P = d.P;
        if (prolong) {
            double rc, rm, rp, du, dv;
            prolong_apply(pc, raw, iu, iv, jv, rc, rm, rp, du, dv);
            v[0] += rc;
            v[1] += rm;
            v[2] += rp;
            if (q.su) v[3] += du;
            if (q.sv) v[4] += dv;
        }
        double *s = T.s + (b * T.S + a) * T_ES;
        tile_put(P, s, q.su, q.sv, v);
        s[T_U2] = s[T_U];
        s[T_V2] = s[T_V];
    }
}
template <bool PJ, int NS, int TS>
__device__ __forceinline__ void fused_body(const Item1 &it, int dir, double omega, int prolong)
{
    typedef Fused<NS, TS> G;
    constexpr int NT = FUSED_BLK(PJ);
    extern __shared__ __attribute__((aligned(16))) double sm[];
    const Desc &d = *it.d;
    int i0, j0; // of the tile
    if (!item_tile_at<TS>(it, 0, d, i0, j0)) return;
    const int par = it_par(it, 0);
    View L = view_of(it, d, par);
    const LevOut o = out_of(it, d, par);
    View O = L; // where the sweep's cell results go
    if (dir) {
        L.c = o.c2; L.mu = o.mu2; L.p = o.p2;
    } else {
        O.c = o.c2; O.mu = o.mu2; O.p = o.p2;
    }
    Tile T;
    T.s = sm; T.i0 = i0 - G::EXT; T.j0 = j0 - G::EXT; T.W = G::W; T.H = G::W; T.S = G::S;
    PSrc ps = {};
    if (prolong) ps = psrc_of(it, d, it_cpar(it, 0));
    const auto &dc = consts_of(it, d);
    fused_load<NT>(dc, L, T, prolong, ps);
    const Phys P = dc.P;
    const Kon<double> K = dc.K;
    const Rhs F = o.F;
    double *const un = o.un, *const vn = o.vn;
    __syncthreads();
    const int hlf = threadIdx.x & 1;
    // a half-sweep of the region widened by ext cells
    auto half = [&](auto cext, auto ccol) {
        constexpr int ext = cext.value, colour = ccol.value, w = TS + 2 * ext;
        for (int pr = threadIdx.x >> 1; pr < w * w / 2; pr += NT / 2) {
            const int lj = pr / (w / 2), kk = pr - lj * (w / 2);
            const int tj = j0 - ext + lj, ti = i0 - ext + 2 * kk + ((tj + colour) & 1);
            if ((L.bcx || (ti >= 0 && ti < L.m1)) && (L.bcy || (tj >= 0 && tj < L.m2))) {
                const int i = L.bcx ? wrapi(ti, L.m1) : ti, j = L.bcy ? wrapi(tj, L.m2) : tj;
                relax_cell<PJ, 1, 1, true>(P, K, L, T, F, nullptr, nullptr, i, j, ti, tj, hlf, omega, 1.0, colour);
            }
        }
        __syncthreads();
    };
    typedef std::integral_constant<int, 0> Red;
    typedef std::integral_constant<int, 1> Black;
    half(std::integral_constant<int, G::EXT>(), Red());
    if (NS == 2) {
        half(std::integral_constant<int, G::EXT - 2>(), Black());
        half(std::integral_constant<int, 2>(), Red());
    }
    if (threadIdx.x < TS * TS) {
        // black cells of the tile: the box faces go to buffer par ^ 1
        const int pr = threadIdx.x >> 1, lj = pr / (TS / 2), kk = pr - lj * (TS / 2);
        const int j = j0 + lj, i = i0 + 2 * kk + ((j + 1) & 1);
        if (i < L.m1 && j < L.m2) relax_cell<PJ, 0, 1, true>(P, K, O, T, F, un, vn, i, j, i, j, hlf, omega, 1.0, 1);
    } else if (threadIdx.x < 2 * TS * TS) {
        // red cells of the tile: their final values
        const int q = (threadIdx.x - TS * TS) >> 1, lj = q / (TS / 2), kk = q - lj * (TS / 2);
        const int j = j0 + lj, i = i0 + 2 * kk + (j & 1);
        if (i < L.m1 && j < L.m2) {
            const double *e = T.at(i, j);
            const size_t g = (size_t)j * L.pitch + i;
            if (hlf == 0) {
                sta<1>(O.c, g, e[T_C]);
                sta<1>(O.mu, g, e[T_MU]);
            } else {
                sta<1>(O.p, g, e[T_P]);
            }
        }
    }
}
template <bool PJ> __device__ __forceinline__ void k_hs_fused_body(const Item1 &it, int dir, double omega, int prolong)
{
    fused_body<PJ, 1, 16>(it, dir, omega, prolong);
}
QN_KERNEL1_PJ(k_hs_fused, __launch_bounds__(FUSED_BLK(PJ)), (int dir, double omega, int prolong), (dir, omega, prolong))
template <bool PJ> __device__ __forceinline__ void k_hs_fused2_body(const Item1 &it, int dir, double omega, int prolong)
{
    fused_body<PJ, 2, 8>(it, dir, omega, prolong);
}
QN_KERNEL1_PJ(k_hs_fused2, __launch_bounds__(FUSED_BLK(PJ)), (int dir, double omega, int prolong), (dir, omega, prolong))

// plain copy, used to measure the copy bandwidth and to calibrate counters
__global__ __launch_bounds__(BLK) void k_copy_probe(const double *__restrict__ a, double *__restrict__ b, size_t n)
{
    for (size_t q = (size_t)blockIdx.x * BLK + threadIdx.x; q < n; q += (size_t)gridDim.x * BLK) b[q] = a[q];
}

// R w of a coarse cell from the values of its four children (a, b: the
// children (0, 0), (1, 0); c, d: (0, 1), (1, 1)): the mean, summed in the order
// k_restrict sums the children's residuals
__device__ __forceinline__ double rw_mean(double a, double b, double c, double d)
{
    return 0.25 * ((a + b) + (c + d));
}

// fine residual r = f - N(w) restricted to the coarse grid together with the
// iterate (cells: mean of the four children; faces: mean of the two coincident
// fine faces), and the FAS right-hand side f_H = N_H(R w) + R r of the coarse
// cells.  A tile of fine cells covers (TX/2) x (TY/2) coarse cells.  One lane per
// fine cell (waves 0-3, a coarse cell's children in a quad of lanes, summed by
// DPP), a fifth wave for the residuals of the tile's 64 coarse cells meanwhile:
// N_H is evaluated on a coarse tile whose halo takes R w from the fine arrays
// directly (the neighbouring workgroups write the coarse iterate meanwhile).
//
// Single-slot elements of 12 values and tiles of only what a residual reads, 18 x
// 18, fit three workgroups in a CU's LDS instead of two: 512 x 2048 cells 52
// instead of 71 us.  (Rows of 20 elements keep a quad's cells on different banks.)
#define RBLK (TBLK + 64)
#define CTILE_S (TX / 2 + 2)
static_assert((TX / 2) * (TY / 2) == 64, "k_restrict: one wave of coarse cells");
// sum over a quad of lanes as (0 + 1) + (2 + 3), the order of rw_mean
__device__ __forceinline__ double quad_sum(double x)
{
    x += other(x);
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), 0x4E, 0xF, 0xF, false),
              hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x4E, 0xF, 0xF, false);
    return x + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <bool PJ, typename IT> __device__ __forceinline__ void k_restrict_body(const IT &it, int set)
{
    TILE_LDS double sm[T_NF * TILE_S * (TY + 2)];
    TILE_LDS double smc[T_NF * CTILE_S * (TY / 2 + 2)];
    __shared__ double part[5][(TX / 2) * (TY / 2)]; // sums of the fine residuals
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    if (!tile_valid(it, k, d)) return;
    const Desc &C = (&d)[1];
    const struct {
        Phys P;
    } dp = { d.P }; // (read at once with the pointers of both levels)
    const int cp = it_cpar(it, k);
    View Lf = view_of(d, it_par(it, k));
    if (set) { // the pre-smoothing left the cells in the second set
        Lf.c = d.c2; Lf.mu = d.mu2; Lf.p = d.p2;
    }
    const View Lc = view_of(C, cp);
    const Tile1 T = item_tile<Tile1, TX + 2>(sm, it, k, d);
    // the coarse tile of R w, from the fine arrays directly (its halo lies
    // in the neighbouring workgroups' tiles), loaded together with the fine
    // tile: cells the mean of the four children, faces the mean of the two
    // coincident fine faces
    Tile1 Tc;
    Tc.s = smc; Tc.i0 = T.i0 / 2; Tc.j0 = T.j0 / 2; Tc.W = TX / 2 + 2; Tc.H = TY / 2 + 2; Tc.S = CTILE_S;
    {
        const int n = Tc.W * Tc.H, e = RBLK - 1 - threadIdx.x;
        const Phys PC = C.P;
        if (e < n) {
            const int bb = e / Tc.W, aa = e - bb * Tc.W;
            const TileSrc s = tile_src(C.m1, C.m2, C.pitch, C.bcx, C.bcy, Tc.i0 - 1 + aa, Tc.j0 - 1 + bb);
            const int Ic = s.c % C.pitch, Jc = s.c / C.pitch;
            const int Iu = s.u % C.pitch, Ju = s.u / C.pitch, Iv = s.v % C.pitch, Jv = s.v / C.pitch;
            const size_t fu = (size_t)(2 * Ju) * Lf.pitch + 2 * Iu, fv = (size_t)(2 * Jv) * Lf.pitch + 2 * Iv;
            // every load before any use (the faces of a wall: loaded in any
            // case, the indices are valid)
            const size_t fa = (size_t)(2 * Jc) * Lf.pitch + 2 * Ic, fb = fa + Lf.pitch;
            const double c4[4] = { lda<1>(Lf.c, fa), lda<1>(Lf.c, fa + 1), lda<1>(Lf.c, fb), lda<1>(Lf.c, fb + 1) };
            const double m4[4] = { lda<1>(Lf.mu, fa), lda<1>(Lf.mu, fa + 1), lda<1>(Lf.mu, fb), lda<1>(Lf.mu, fb + 1) };
            const double p4[4] = { lda<1>(Lf.p, fa), lda<1>(Lf.p, fa + 1), lda<1>(Lf.p, fb), lda<1>(Lf.p, fb + 1) };
            const double u0 = lda<1>(Lf.u, fu), u1 = lda<1>(Lf.u, fu + Lf.pitch);
            const double w0 = lda<1>(Lf.v, fv), w1 = lda<1>(Lf.v, fv + 1);
            const double cn = lda<1>(C.cn, s.c), un = lda<1>(C.un, s.u), vn = lda<1>(C.vn, s.v);
            __builtin_amdgcn_sched_barrier(0);
            if (s.sc == 0) {
                tile_zero(Tc, bb * CTILE_S + aa);
            } else {
                const double w[8] = { rw_mean(c4[0], c4[1], c4[2], c4[3]), rw_mean(m4[0], m4[1], m4[2], m4[3]),
                                      rw_mean(p4[0], p4[1], p4[2], p4[3]), 0.5 * (u0 + u1), 0.5 * (w0 + w1), cn, un, vn };
                tile_put(PC, Tc.s + (bb * CTILE_S + aa) * T_NF, s.su, s.sv, w);
            }
        }
    }
    tile_load<2, RBLK>(dp, Lf, T);
    __syncthreads();
    const bool fine = threadIdx.x < TBLK;
    const int cc = fine ? (int)threadIdx.x >> 2 : (int)threadIdx.x - TBLK, ch = threadIdx.x & 3;
    const int I = Tc.i0 + cc % (TX / 2), J = Tc.j0 + cc / (TX / 2);
    const bool on = I < C.m1 && J < C.m2;
    Resid r = {};
    if (fine) {
        if (on) r = resid_cell<PJ>(d.K, Lf, T, rhs_of(d), 2 * I + (ch & 1), 2 * J + (ch >> 1));
        // the faces of the coarse cell: west faces of the children (0, .),
        // south faces of the children (., 0)
        const double sc = quad_sum(r.c), smu = quad_sum(r.mu), sp = quad_sum(r.p),
                     su = quad_sum(ch & 1 ? 0.0 : r.u), sv = quad_sum(ch >> 1 ? 0.0 : r.v);
        if (ch == 0) {
            part[0][cc] = sc; part[1][cc] = smu; part[2][cc] = sp; part[3][cc] = su; part[4][cc] = sv;
        }
    } else if (on) {
        const Rhs Z = { nullptr, nullptr, nullptr, nullptr, nullptr };
        r = resid_cell<PJ>(C.K, Lc, Tc, Z, I, J); // -N_H(R w)
    }
    __syncthreads();
    if (fine || !on) return;
    // the fifth wave: f_H = N_H(R w) + R r on the coarse cells
    const size_t q = (size_t)J * C.pitch + I;
    const double *t = Tc.at(I, J);
    sta<1>(C.c, q, t[T_C]); sta<1>(C.c0, q, t[T_C]);
    sta<1>(C.mu, q, t[T_MU]); sta<1>(C.mu0, q, t[T_MU]);
    sta<1>(C.p, q, t[T_P]); sta<1>(C.p0, q, t[T_P]);
    sta<1>(C.ub[cp], q, t[T_U]); sta<1>(C.u0, q, t[T_U]);
    sta<1>(C.vb[cp], q, t[T_V]); sta<1>(C.v0, q, t[T_V]);
    sta<1>(C.fc, q, 0.25 * part[0][cc] - r.c);
    sta<1>(C.fmu, q, 0.25 * part[1][cc] - r.mu);
    sta<1>(C.fp, q, 0.25 * part[2][cc] - r.p);
    sta<1>(C.fu, q, u_unk(Lc, I) ? 0.5 * part[3][cc] - r.u : 0.0);
    sta<1>(C.fv, q, v_unk(Lc, J) ? 0.5 * part[4][cc] - r.v : 0.0);
}
QN_KERNEL_PJ(k_restrict, __launch_bounds__(RBLK), (int set), (set))

// --------------------------------------------------------------------------
// The bottom of a V-cycle: a level and every coarser one in one workgroup per
// item, resident in LDS: pre-smoothing and restriction down to the coarsest
// level, its solve, prolongation and post-smoothing back up, with the
// arithmetic of the kernels that do the same level by level.  Such levels have
// fewer cells of a colour than a workgroup has lane pairs, so a launch lasts as
// long as its dependent chain; a launch per step also paid for its start (two
// memory round trips), for the level's way from and to memory and for an
// image map of the whole tile.  Per cycle of the 256 x 512 droplet (16 x 32, 8 x 16,
// 4 x 8 cells: 24 half-sweeps), five smoothing launches of 20.8 us and two restrictions of
// 6.4 us became one launch of 61 us (MI355X).
//
// LDS of a level: its tile (rows of an even number of elements), the
// right-hand sides, the restricted iterate (coarser levels), the images.
#define BOT 512
struct BotLev {
    double *f, *w0; // 5 fields of m1*m2
    Image *ring;
    Tile T;
    int m1, m2;
};
__host__ __device__ inline int bot_stride(int m1) { return (m1 + 4) & ~1; }
__host__ __device__ inline size_t bot_tile(int m1, int m2, int es) { return (size_t)es * bot_stride(m1) * (m2 + 3); }
__host__ __device__ inline size_t bot_doubles(int m1, int m2)
{
    return bot_tile(m1, m2, T_ES) + (size_t)10 * m1 * m2 + 2 * (size_t)ring_size(m1, m2);
}
// (the top level has no restricted iterate: the levels' LDS starts that much
// before it)
__host__ __device__ inline size_t bot_skip(int m1, int m2) { return (size_t)5 * m1 * m2; }
// level l below the m1 x m2 one whose LDS starts at sm
__device__ __forceinline__ BotLev bot_lev(double *sm, int m1, int m2, int l)
{
    const bool top = l == 0;
    int off = top ? 0 : -(int)(bot_skip(m1, m2) / 2); // in 16 bytes (el)
    for (; l > 0; l--) {
        off += (int)(bot_doubles(m1, m2) / 2);
        m1 >>= 1;
        m2 >>= 1;
    }
    sm += 2 * off;
    BotLev B;
    B.m1 = m1; B.m2 = m2;
    B.T.s = sm; B.T.i0 = 0; B.T.j0 = 0; B.T.W = m1 + 3; B.T.H = m2 + 3; B.T.S = bot_stride(m1);
    B.f = sm + bot_tile(m1, m2, T_ES);
    B.w0 = B.f + 5 * m1 * m2;
    B.ring = (Image *)(top ? B.w0 : B.w0 + 5 * m1 * m2);
    return B;
}
// item e of the items of levels l, l + 1, .. of `depth`, size(m1, m2) on each:
// its level and its place there; whether there is one
template <typename F> __device__ __forceinline__ bool bot_find(int &l, int &e, int depth, int m1, int m2, F size)
{
    for (; l < depth; l++) {
        const int n = size(m1 >> l, m2 >> l);
        if (e < n) return true;
        e -= n;
    }
    return false;
}
// f(lev(l), k) for the ring entries k of every level l
template <typename L, typename F> __device__ __forceinline__ void bot_rings(int depth, int m1, int m2, L lev, F f)
{
    for (int e = threadIdx.x;; e += BOT) {
        int l = 0, k = e;
        if (!bot_find(l, k, depth, m1, m2, ring_size)) break;
        f(lev(l), k);
    }
}
__device__ __forceinline__ View bot_view(const BotLev &B, const Desc &d)
{
    View L = {};
    L.m1 = B.m1; L.m2 = B.m2; L.pitch = B.m1;
    L.bcx = d.bcx; L.bcy = d.bcy;
    return L;
}
__device__ __forceinline__ Rhs bot_rhs(const BotLev &B)
{
    const int n = B.m1 * B.m2;
    const Rhs F = { B.f, B.f + n, B.f + 2 * n, B.f + 3 * n, B.f + 4 * n };
    return F;
}
// the images follow their sources, for a residual (relaxations read the sources)
// (thread t of BOT)
__device__ __forceinline__ void bot_images(const BotLev &B, int t)
{
    const int n = ring_size(B.m1, B.m2);
    for (int k = t; k < n; k += BOT) {
        const Image g = B.ring[k];
        const double *s = B.T.s + g.c * T_ES;
        const double c = s[T_C], mu = s[T_MU], p = s[T_P], rs = s[T_RS];
        const double u = B.T.s[(g.u >> 2) * T_ES + T_U], v = B.T.s[(g.v >> 2) * T_ES + T_V];
        double *t = B.T.s + g.e * T_ES;
        t[T_C] = c;
        t[T_MU] = mu;
        t[T_P] = p;
        t[T_RS] = rs;
        t[T_U] = signed_val((g.u & 3) - 1, u);
        t[T_V] = signed_val((g.v & 3) - 1, v);
    }
}
// sweeps of a level (an even number of half-sweeps: the faces end in slot 0)
template <bool PJ>
__device__ __forceinline__ void bot_smooth(const Phys &P, const Desc &d, const BotLev &B, int sweeps, double omega, double pomega)
{
    const Kon<double> K = d.K;
    const View L = bot_view(B, d);
    const Rhs F = bot_rhs(B);
    // a thread's first cell of a sweep (a level of more cells of a colour
    // than lane pairs takes several passes)
    const int half = B.m1 >> 1, n2 = 2 * half * B.m2, pr = threadIdx.x >> 1, hlf = threadIdx.x & 1;
    const int j0 = pr / half, i0 = 2 * (pr - j0 * half), dj = (BOT / 2) / half, di = 2 * ((BOT / 2) - dj * half);
    auto sweep = [&](auto colour) {
        int i = i0, j = j0;
        for (int t = threadIdx.x; t < n2; t += BOT) {
            const int ic = i + ((j + colour.value) & 1);
            relax_cell<PJ, 2, 3, true>(P, K, L, B.T, F, nullptr, nullptr, ic, j, ic, j, hlf, omega, pomega, colour.value);
            i += di;
            j += dj;
            if (i >= B.m1) { i -= B.m1; j++; }
        }
        __syncthreads();
    };
    for (int s = 0; s < sweeps; s++) {
        sweep(std::integral_constant<int, 0>());
        sweep(std::integral_constant<int, 1>());
    }
}
// residual of level A, restricted with the iterate to the next level C, whose
// right-hand side becomes N_H(R w) + R r
template <bool PJ>
__device__ __forceinline__ void bot_restrict(const Phys &P, const Desc &d, const BotLev &A, const BotLev &C)
{
    const int nc = C.m1 * C.m2, rt = BOT - 1 - threadIdx.x;
    // R w, by the last threads, while the first ones update the images of A
    for (int t = rt; t < nc; t += BOT) {
        const int J = t / C.m1, I = t - J * C.m1;
        const double *a = A.T.at(2 * I, 2 * J), *b = a + T_ES, *s = el<T_ES>(a, A.T.S), *e = s + T_ES;
        const double w[5] = { 0.25 * ((a[T_C] + b[T_C]) + (s[T_C] + e[T_C])), 0.25 * ((a[T_MU] + b[T_MU]) + (s[T_MU] + e[T_MU])),
                              0.25 * ((a[T_P] + b[T_P]) + (s[T_P] + e[T_P])), 0.5 * (a[T_U] + s[T_U]),
                              0.5 * (a[T_V] + b[T_V]) };
        double *o = C.T.at(I, J);
        o[T_C] = w[0];
        o[T_MU] = w[1];
        o[T_P] = w[2];
        o[T_RS] = rho_of(P, w[0]);
        o[T_U] = o[T_U2] = w[3];
        o[T_V] = o[T_V2] = w[4];
#pragma unroll
        for (int q = 0; q < 5; q++) C.w0[q * nc + t] = w[q];
    }
    bot_images(A, threadIdx.x);
    __syncthreads();
    // R r; the images of C meanwhile
    {
        const Kon<double> K = d.K;
        const View L = bot_view(A, d);
        const Rhs F = bot_rhs(A);
        bot_images(C, rt);
        for (int t = threadIdx.x; t < 4 * nc; t += BOT) {
            const int cc = t >> 2, ch = t & 3;
            const int J = cc / C.m1, I = cc - J * C.m1, i = 2 * I + (ch & 1), j = 2 * J + (ch >> 1);
            const Resid r = resid_cell<PJ, 3>(K, L, A.T, F, i, j);
            const bool wu = (ch & 1) == 0, wv = (ch >> 1) == 0; // faces of the coarse cell
            const double f[5] = { 0.25 * quad_sum(r.c), 0.25 * quad_sum(r.mu), 0.25 * quad_sum(r.p),
                                  0.5 * quad_sum(wu ? r.u : 0.0), 0.5 * quad_sum(wv ? r.v : 0.0) };
            if (ch == 0)
#pragma unroll
                for (int q = 0; q < 5; q++) C.f[q * nc + cc] = f[q];
        }
    }
    __syncthreads();
    {
        const Desc &dc = (&d)[1];
        const Kon<double> K = dc.K;
        const View L = bot_view(C, dc);
        const Rhs Z = { nullptr, nullptr, nullptr, nullptr, nullptr };
        for (int t = threadIdx.x; t < nc; t += BOT) {
            const int J = t / C.m1, I = t - J * C.m1;
            const Resid r = resid_cell<PJ, 3>(K, L, C.T, Z, I, J); // -N_H(R w)
            C.f[t] -= r.c;
            C.f[nc + t] -= r.mu;
            C.f[2 * nc + t] -= r.p;
            C.f[3 * nc + t] -= r.u;
            C.f[4 * nc + t] -= r.v;
        }
    }
    __syncthreads();
}
// the coarse-grid correction (k_prolong's arithmetic) from level C to A
__device__ __forceinline__ void bot_prolong(const Phys &P, const Desc &d, const BotLev &A, const BotLev &C)
{
    const int na = A.m1 * A.m2, nc = C.m1 * C.m2;
    const bool bx = d.bcx, by = d.bcy;
    for (int t = threadIdx.x; t < na; t += BOT) {
        const int j = t / A.m1, i = t - j * A.m1, I = i >> 1, J = j >> 1;
        auto corr = [&](int f, int a, int b) { return C.T.at(a, b)[f] - C.w0[(f == T_C ? 0 : f == T_MU ? 1 : f == T_P ? 2 : f == T_U ? 3 : 4) * nc + b * C.m1 + a]; };
        // (no loads under a condition: they would wait for each other)
        const bool ix = I + 1 < C.m1, jy = J + 1 < C.m2;
        const double u0 = corr(T_U, I, J), u1 = corr(T_U, ix ? I + 1 : 0, J), v0 = corr(T_V, I, J),
                     v1 = corr(T_V, I, jy ? J + 1 : 0);
        const double du = i & 1 ? 0.5 * (u0 + (ix || bx ? u1 : 0.0)) : u0, dv = j & 1 ? 0.5 * (v0 + (jy || by ? v1 : 0.0)) : v0;
        double *o = A.T.at(i, j);
        const double c = o[T_C] + corr(T_C, I, J);
        o[T_C] = c;
        o[T_MU] += corr(T_MU, I, J);
        o[T_P] += corr(T_P, I, J);
        o[T_RS] = rho_of(P, c);
        if (bx || i >= 1) o[T_U] += du;
        if (by || j >= 1) o[T_V] += dv;
    }
    __syncthreads();
}
template <bool PJ, typename IT>
__device__ __forceinline__ void k_bottom_body(const IT &it, int nu1, int nu2, int nuc, double omega, double comega)
{
    extern __shared__ __attribute__((aligned(16))) double sm[];
    const int k = find_item(it);
    if ((int)blockIdx.x != it_start(it, k)) return; // pads the list: the levels are one workgroup's, in place
    const Desc &d = it_desc(it, k);
    const Phys P = d.P;
    const int par = it_par(it, k), m1 = d.m1, m2 = d.m2, depth = d.depth;
    const View L = view_of(d, par);
    double *const ua = d.ub[par], *const va = d.vb[par];
    // The cells of the top level with their right-hand sides, and the time-n data
    // of the coarser levels' cells (no more than BOT in all), every load before
    // any use; the images' sources meanwhile, and then the images' time-n data.
    const int n = m1 * m2;
    int lc = 1, ec = threadIdx.x;
    const bool hc = bot_find(lc, ec, depth, m1, m2, [](int a, int b) { return a * b; });
    auto lev = [&](int l) { return bot_lev(sm, m1, m2, l); };
    const BotLev Bc = lev(hc ? lc : 0);
    const int jc = ec / Bc.m1, ic = ec - jc * Bc.m1;
    const Desc &dc = (&d)[hc ? lc : 0];
    const double *const pc = dc.cn, *const pu = dc.un, *const pv = dc.vn;
    {
        const Rhs F = rhs_of(d);
        const BotLev B = bot_lev(sm, m1, m2, 0);
        for (int t0 = threadIdx.x; t0 < n || t0 < BOT; t0 += BOT) {
            const int e = min(t0, n - 1), j = e / m1, i = e - j * m1;
            const TileSrc q = tile_src(m1, m2, L.pitch, L.bcx, L.bcy, i, j);
            const double v[8] = { lda<1>(L.c, q.c), lda<1>(L.mu, q.c), lda<1>(L.p, q.c), lda<1>(L.u, q.u),
                                  lda<1>(L.v, q.v), lda<1>(L.cn, q.c), lda<1>(L.un, q.u), lda<1>(L.vn, q.v) };
            double f[5] = { 0.0, 0.0, 0.0, 0.0, 0.0 };
            if (F.fc) {
                f[0] = lda<1>(F.fc, q.c); f[1] = lda<1>(F.fmu, q.c); f[2] = lda<1>(F.fp, q.c);
                f[3] = lda<1>(F.fu, q.c); f[4] = lda<1>(F.fv, q.c);
            }
            const bool co = hc && t0 < BOT;
            double w[3] = { 0.0, 0.0, 0.0 };
            TileSrc qc = {};
            if (co) {
                qc = tile_src(Bc.m1, Bc.m2, Bc.m1, L.bcx, L.bcy, ic, jc);
                w[0] = lda<1>(pc, qc.c); w[1] = lda<1>(pu, qc.u); w[2] = lda<1>(pv, qc.v);
            }
            if (t0 < BOT)
                bot_rings(depth, m1, m2, lev, [&](const BotLev &R, int k) { R.ring[k] = ring_entry(R.T, R.m1, R.m2, L.bcx, L.bcy, k); });
            __builtin_amdgcn_sched_barrier(0);
            if (t0 < n) {
                double *t = B.T.at(i, j);
                tile_put(P, t, q.su, q.sv, v);
                t[T_U2] = t[T_U];
                t[T_V2] = t[T_V];
#pragma unroll
                for (int g = 0; g < 5; g++) B.f[g * n + e] = f[g];
            }
            if (co) {
                double *o = Bc.T.at(ic, jc);
                o[T_CN] = w[0];
                o[T_RN] = rho_of(P, w[0]);
                o[T_MV] = visc_of(P, w[0]);
                o[T_MOB] = mob_of(P, w[0]);
                o[T_UN] = signed_val(qc.su, w[1]);
                o[T_VN] = signed_val(qc.sv, w[2]);
            }
        }
    }
    __syncthreads();
    bot_rings(depth, m1, m2, lev, [&](const BotLev &R, int k) {
        const Image g = R.ring[k];
        const double *s = R.T.s + g.c * T_ES;
        const double cn = s[T_CN], rn = s[T_RN], mv = s[T_MV], mb = s[T_MOB], un = R.T.s[(g.u >> 2) * T_ES + T_UN],
                     vn = R.T.s[(g.v >> 2) * T_ES + T_VN];
        double *t = R.T.s + g.e * T_ES;
        t[T_CN] = cn;
        t[T_RN] = rn;
        t[T_MV] = mv;
        t[T_MOB] = mb;
        t[T_UN] = signed_val((g.u & 3) - 1, un);
        t[T_VN] = signed_val((g.v & 3) - 1, vn);
        t[T_U] = t[T_U2] = t[T_V] = t[T_V2] = 0.0; // on the faces of a high wall
    });
    __syncthreads();
    // down to the coarsest level and back up (one copy of the code of each
    // phase: it is fetched once).  The coarsest level over-relaxes the velocity
    // and pressure updates (the primitive box, the projection pressure step).
    for (int p = 0; p < 2 * depth - 1; p++) {
        const int l = p < depth ? p : 2 * depth - 2 - p;
        const BotLev B = bot_lev(sm, m1, m2, l);
        if (p > 0 && p < depth) bot_restrict<PJ>(P, (&d)[l - 1], bot_lev(sm, m1, m2, l - 1), B);
        if (p >= depth) bot_prolong(P, d, B, bot_lev(sm, m1, m2, l + 1));
        const bool last = p == depth - 1;
        bot_smooth<PJ>(P, (&d)[l], B, last ? nuc : p < depth ? nu1 : nu2, last && !PJ ? comega : omega, last && PJ ? comega : 1.0);
    }
    const BotLev B = bot_lev(sm, m1, m2, 0);
    for (int e = threadIdx.x; e < m1 * m2; e += BOT) {
        const int j = e / m1, i = e - j * m1;
        const size_t q = (size_t)j * L.pitch + i;
        const double *t = B.T.at(i, j);
        sta<1>(L.c, q, t[T_C]);
        sta<1>(L.mu, q, t[T_MU]);
        sta<1>(L.p, q, t[T_P]);
        sta<1>(ua, q, t[T_U]);
        sta<1>(va, q, t[T_V]);
    }
}
QN_KERNEL_PJ(k_bottom, __launch_bounds__(BOT), (int nu1, int nu2, int nuc, double omega, double comega), (nu1, nu2, nuc, omega, comega))

// w_h += P(w_H - R w_h) on the level the item names, one thread per fine cell
template <typename IT> __device__ __forceinline__ void k_prolong_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const Desc &C = (&d)[1];
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= d.m1 * d.m2) return;
    const int j = t / d.m1, i = t - j * d.m1;
    const size_t kf = (size_t)j * d.pitch + i;
    // the correction of the cell and its west and south faces, every load
    // issued before any use
    const PSrc ps = psrc_of(d, &C, it_cpar(it, k));
    double *ub = d.ub[it_par(it, k)], *vb = d.vb[it_par(it, k)];
    const PRaw raw = prolong_load(ps, i, j, i, j, i, j);
    const double c = lda<1>(d.c, kf), mu = lda<1>(d.mu, kf), p = lda<1>(d.p, kf), u = lda<1>(ub, kf),
                 v = lda<1>(vb, kf);
    __builtin_amdgcn_sched_barrier(0);
    double rc, rm, rp, du, dv;
    prolong_apply(ps, raw, i, i, j, rc, rm, rp, du, dv);
    sta<1>(d.c, kf, c + rc);
    sta<1>(d.mu, kf, mu + rm);
    sta<1>(d.p, kf, p + rp);
    if (ps.bcx || i >= 1) sta<1>(ub, kf, u + du);
    if (ps.bcy || j >= 1) sta<1>(vb, kf, v + dv);
}
QN_KERNEL(k_prolong, __launch_bounds__(BLK), (), ())

// Sums over the block of its threads' first N values (a power of two), through
// N * NT doubles of LDS that nothing else holds any more: a value's NT terms
// are added by NT / N threads each, in a fixed order.  Against a reduction in
// registers (shuffles and selects of all NRED values: 380 of the residual
// norms' 970 vector instructions per wave) the norms of 2048 x 2048 cells took 103
// instead of 146 us.
template <int NT, int N> __device__ __forceinline__ void block_sum_lds(const double (&v)[NRED], double *sm, double *out, int st)
{
    constexpr int G = NT / N; // threads per value
    static_assert(G <= 64 && G >= 16 && NT % (2 * G) == 0, "block_sum_lds");
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; q++) sm[q * NT + threadIdx.x] = v[q];
    __syncthreads();
    const int q = threadIdx.x / G, g = threadIdx.x % G;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NT; k += 2 * G) {
        const double *p = sm + q * NT + k + 2 * g;
        s += p[0] + p[1];
    }
    for (int m = 1; m < G; m <<= 1) s += __shfl_xor(s, m, 64);
    if (g == 0) out[(size_t)q * st] = s;
    if (N < NRED && threadIdx.x >= N && threadIdx.x < NRED) out[(size_t)threadIdx.x * st] = 0.0;
}
// wave64 + LDS block sum of NRED values (blocks of NT threads).  Within a
// wave each exchange halves the number of slots a lane is responsible for
// (lane l ends with the sum of slot l / 4): 17 exchanges instead of 6 per slot.
template <int NT> __device__ __forceinline__ void block_sum_store(double (&v)[NRED], double *out, int st)
{
    static_assert(NRED == 16, "block_sum_store");
    __shared__ double sh[NT / 64][NRED];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    double a[8];
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const bool h = l & 32;
        a[q] = (h ? v[q + 8] : v[q]) + __shfl_xor(h ? v[q] : v[q + 8], 32, 64);
    }
#pragma unroll
    for (int n = 4; n > 0; n >>= 1) {
        const bool h = l & (4 * n);
#pragma unroll
        for (int q = 0; q < n; q++) a[q] = (h ? a[q + n] : a[q]) + __shfl_xor(h ? a[q] : a[q + n], 4 * n, 64);
    }
    a[0] += __shfl_xor(a[0], 2, 64);
    a[0] += __shfl_xor(a[0], 1, 64);
    if ((l & 3) == 0) sh[w][l >> 2] = a[0];
    __syncthreads();
    if (threadIdx.x < NRED) {
        double s = 0.0;
        for (int ww = 0; ww < NT / 64; ww++) s += sh[ww][threadIdx.x];
        out[(size_t)threadIdx.x * st] = s;
    }
}

// Acceleration of the cycle iteration, recording of a cycle result in ring
// slot s = ac & 15: the residual and the iterate of the cell at index w and
// its west and south faces, and the cell's share of the normal equations of
// min || r + sum_a g_a (r - r_a) ||, r_a the residual a + 1 slots back
// (a < np = ac >> 4): v[7 + b(b+1)/2 + a] += e_a e_b (a <= b), v[13 + a] += e_a r,
// e_a = r - r_a.  Every earlier residual is loaded before any store or
// product.
__device__ __forceinline__ void acc_record(const Desc &d, int ac, size_t w, const Resid &r, const double *t,
                                           double (&v)[NRED])
{
    const int s = ac & 15, np = ac >> 4, R = d.am;
    const size_t st = (size_t)d.pitch * d.m2;
    double *const ar = d.ar, *const aw = d.aw;
    const double x[5] = { r.c, r.mu, r.p, r.u, r.v }, y[5] = { t[T_C], t[T_MU], t[T_P], t[T_U], t[T_V] };
    double old[3][5];
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
        for (int f = 0; f < 5; f++)
            old[a][f] = a < np ? lda<1>(ar, (size_t)(((s - 1 - a + R) % R) * 5 + f) * st + w) : 0.0;
#pragma unroll
    for (int f = 0; f < 5; f++) {
        sta<1>(ar, (size_t)(s * 5 + f) * st + w, x[f]);
        sta<1>(aw, (size_t)(s * 5 + f) * st + w, y[f]);
    }
#pragma unroll
    for (int f = 0; f < 5; f++) {
        double e[3];
#pragma unroll
        for (int a = 0; a < 3; a++) e[a] = a < np ? x[f] - old[a][f] : 0.0;
#pragma unroll
        for (int b = 0; b < 3; b++)
#pragma unroll
            for (int a = 0; a <= b; a++) v[7 + b * (b + 1) / 2 + a] += e[a] * e[b];
#pragma unroll
        for (int a = 0; a < 3; a++) v[13 + a] += e[a] * x[f];
    }
}

// residual norms of a finest level: per tile sums of r^2 for the five
// equations, the sum of pbar, and the count of cells that are non-finite or
// past the density pole (partials indexed by the tile's place in the band
// order); optionally the residual fields themselves.  One lane per cell.
template <bool PJ, typename IT> __device__ __forceinline__ void k_resid_norm_body(const IT &it)
{
    TILE_LDS double sm[NRED * TBLK]; // the tile, then the sums
    static_assert(T_NF * (TX + 2) * (TY + 2) <= NRED * TBLK, "k_resid_norm");
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    if (!tile_valid(it, k, d)) return;
    const int par = it_par(it, k);
    const View L = view_of(it, d, par);
    const Tile1 T = item_tile<Tile1, TX + 2, TX + 2>(sm, it, k, d);
    const auto &dc = consts_of(it, d);
    tile_load<2, TBLK>(dc, L, T);
    const Phys P = dc.P;
    const Kon<double> K = dc.K;
    __syncthreads();
    double v[NRED] = {};
    const size_t n = (size_t)L.m1 * L.m2;
    const int i = T.i0 + (int)threadIdx.x % TX, j = T.j0 + (int)threadIdx.x / TX;
    if (i < L.m1 && j < L.m2) {
        const Resid r = resid_cell<PJ>(K, L, T, rhs_of(d), i, j);
        const double *t = T.at(i, j);
        const double c = t[T_C], pp = t[T_P];
        v[0] = r.c * r.c;
        v[1] = r.mu * r.mu;
        v[2] = r.p * r.p;
        v[3] = r.u * r.u;
        v[4] = r.v * r.v;
        v[5] = pp;
        const bool ok = isfinite(c) && isfinite(t[T_MU]) && isfinite(pp) && isfinite(t[T_U]) && isfinite(t[T_V])
                      && (P.drho * c + P.rho1 > 0.0);
        v[6] = ok ? 0.0 : 1.0;
        const size_t q = (size_t)j * L.m1 + i, w = (size_t)j * L.pitch + i;
        if (d.rout) {
            d.rout[q] = r.c;
            d.rout[n + q] = r.mu;
            d.rout[2 * n + q] = r.p;
            d.rout[3 * n + q] = r.u;
            d.rout[4 * n + q] = r.v;
        }
        if (d.rc) {
            // mixed precision: the right-hand side and linearisation point of
            // the next correction cycle, whose correction starts at zero
            d.rc[w] = (float)r.c; d.rmu[w] = (float)r.mu; d.rp[w] = (float)r.p; d.ru[w] = (float)r.u; d.rv[w] = (float)r.v;
            d.xc[w] = (float)c; d.xmu[w] = (float)t[T_MU]; d.xu[w] = (float)t[T_U]; d.xv[w] = (float)t[T_V];
            d.dc[w] = 0.0f; d.dmu[w] = 0.0f; d.dp[w] = 0.0f; d.dub[par][w] = 0.0f; d.dvb[par][w] = 0.0f;
        }
        const int ac = it_acc(it, k);
        if (ac >= 0 && d.ar) acc_record(d, ac, w, r, t, v);
    }
    const int tl = (T.j0 / TY) * it_cnt(it, k) + T.i0 / TX;
    double *const out = d.partials + tl;
    const int st = part_stride(d);
    if (it_acc(it, k) >= 0 && d.ar) block_sum_lds<TBLK, NRED>(v, sm, out, st);
    else block_sum_lds<TBLK, 8>(v, sm, out, st);
}
QN_KERNEL_PJ(k_resid_norm, __launch_bounds__(TBLK), (), ())

// mass and energy partial sums of the current state, one thread per cell
template <typename IT> __device__ __forceinline__ void k_mass_energy_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const View L = view_of(d, it_par(it, k));
    const Phys &P = d.P;
    const int b = (int)blockIdx.x - it_start(it, k);
    if (b * BLK >= d.m1 * d.m2) return; // pads the list: no partials of its own
    const int t = b * BLK + threadIdx.x;
    double v[NRED] = {};
    if (t < L.m1 * L.m2) {
        const int j = t / L.m1, i = t - j * L.m1;
        const size_t q = (size_t)j * L.pitch + i;
        const double c = L.c[q], r = rho_of(P, c);
        v[0] = r * c;
        v[1] = r * (1.0 - c);
        const double cw = ldc(L.c, L.m1, L.m2, L.pitch, L.bcx, L.bcy, i - 1, j);
        const double cs = ldc(L.c, L.m1, L.m2, L.pitch, L.bcx, L.bcy, i, j - 1);
        const double rw = rho_of(P, cw), rs = rho_of(P, cs);
        // kinetic energy on the west and south faces of the cell (App. A.7)
        if (u_unk(L, i)) { const double u = L.u[q]; v[2] += 0.25 * (r + rw) * u * u; }
        if (v_unk(L, j)) { const double w = L.v[q]; v[2] += 0.25 * (r + rs) * w * w; }
        // gradient energy [rho D c, D c] on the same faces (walls carry none)
        if (L.bcx || i > 0) { const double g = (c - cw) * L.inv_h; v[3] += 0.5 * (r + rw) * g * g; }
        if (L.bcy || j > 0) { const double g = (c - cs) * L.inv_h; v[3] += 0.5 * (r + rs) * g * g; }
        v[4] = r * dwell(c);
        v[5] = (r - P.rho_ref) * (j + 0.5) * d.h;
    }
    block_sum_store<BLK>(v, d.partials + b, part_stride(d));
}
QN_KERNEL(k_mass_energy, __launch_bounds__(BLK), (), ())

// Dissipation of the step just taken (Theorem of sec. 6.1 with the norms of
// App. A.7), from the new iterate and the time-n data still held by the
// level: partial sums, per cell, of
//   0: mu(c^n) (|d_x u|^2 + |d_y v|^2 + 1/4 sum over the 4 corners of
//      |calD_y u|^2 + |calD_x v|^2)        (viscous gradient norm)
//   1: mu(c^n) (d_x u + d_y v)^2           (viscous divergence norm)
//   2: A m(c^n) |D mu_c|^2 on the west and south faces, mu_c = mubar + alpha pbar
//   3: A rho^n |u - u^n|^2 on the west and south faces (unknown faces only)
// One thread per cell.
template <typename IT> __device__ __forceinline__ void k_dissipation_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    // projection scheme: the viscous parts and the time-difference part are
    // taken on the intermediate velocity (the other face buffer), and slot 4
    // sums A rho(c) (u^{n+1} - u~)^2 over the faces
    const bool pj = d.P.scheme != 0;
    const View L = view_of(d, pj ? it_par(it, k) ^ 1 : it_par(it, k));
    const double *uf = d.ub[it_par(it, k)], *vf = d.vb[it_par(it, k)];
    const Phys &P = d.P;
    const int b = (int)blockIdx.x - it_start(it, k);
    if (b * BLK >= d.m1 * d.m2) return; // pads the list: no partials of its own
    const int t = b * BLK + threadIdx.x;
    double v[NRED] = {};
    if (t < L.m1 * L.m2) {
        const int j = t / L.m1, i = t - j * L.m1;
        const int m1 = L.m1, m2 = L.m2, pt = L.pitch, bx = L.bcx, by = L.bcy;
        const double ih = L.inv_h;
        auto U = [&](int a, int c) { return ldu(L.u, m1, m2, pt, bx, by, a, c); };
        auto V = [&](int a, int c) { return ldv(L.v, m1, m2, pt, bx, by, a, c); };
        auto CN = [&](int a, int c) { return ldc(L.cn, m1, m2, pt, bx, by, a, c); };
        const double mv = visc_of(P, CN(i, j));
        const double dxu = (U(i + 1, j) - U(i, j)) * ih, dyv = (V(i, j + 1) - V(i, j)) * ih;
        double sv = 0.0;
#pragma unroll
        for (int a = 0; a <= 1; a++)
#pragma unroll
            for (int c = 0; c <= 1; c++) {
                const double dyu = (U(i + a, j + c) - U(i + a, j + c - 1)) * ih;
                const double dxv = (V(i + a, j + c) - V(i + a - 1, j + c)) * ih;
                sv += dyu * dyu + dxv * dxv;
            }
        v[0] = mv * (dxu * dxu + dyv * dyv + 0.25 * sv);
        v[1] = mv * (dxu + dyv) * (dxu + dyv);
        const double c0 = CN(i, j), mob0 = mob_of(P, c0), r0 = rho_of(P, c0);
        const double mu0 = ldc(L.mu, m1, m2, pt, bx, by, i, j), p0 = ldc(L.p, m1, m2, pt, bx, by, i, j);
        const size_t q = (size_t)j * pt + i;
        if (bx || i > 0) {
            const double cw = CN(i - 1, j);
            const double g = (mu0 - ldc(L.mu, m1, m2, pt, bx, by, i - 1, j)) * ih
                           + P.alpha * (p0 - ldc(L.p, m1, m2, pt, bx, by, i - 1, j)) * ih;
            v[2] += 0.5 * (mob0 + mob_of(P, cw)) * g * g;
            const double du = L.u[q] - L.un[q];
            v[3] += 0.5 * (r0 + rho_of(P, cw)) * du * du;
            if (pj) {
                const double dp = uf[q] - L.u[q];
                v[4] += 0.5 * (rho_of(P, L.c[q]) + rho_of(P, ldc(L.c, m1, m2, pt, bx, by, i - 1, j))) * dp * dp;
            }
        }
        if (by || j > 0) {
            const double cs = CN(i, j - 1);
            const double g = (mu0 - ldc(L.mu, m1, m2, pt, bx, by, i, j - 1)) * ih
                           + P.alpha * (p0 - ldc(L.p, m1, m2, pt, bx, by, i, j - 1)) * ih;
            v[2] += 0.5 * (mob0 + mob_of(P, cs)) * g * g;
            const double dv = L.v[q] - L.vn[q];
            v[3] += 0.5 * (r0 + rho_of(P, cs)) * dv * dv;
            if (pj) {
                const double dp = vf[q] - L.v[q];
                v[4] += 0.5 * (rho_of(P, L.c[q]) + rho_of(P, ldc(L.c, m1, m2, pt, bx, by, i, j - 1))) * dp * dp;
            }
        }
    }
    block_sum_store<BLK>(v, d.partials + b, part_stride(d));
}
QN_KERNEL(k_dissipation, __launch_bounds__(BLK), (), ())

// Projection scheme, end of a converged step: the velocity of time n+1 from
// the projection equation (pj-num-pjx) (as face_final) on every west and
// south face, written to the other face buffer, which becomes the current
// one; the intermediate velocity stays in buffer par for the dissipation.
template <typename IT> __device__ __forceinline__ void k_pj_final_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int par = it_par(it, k);
    const View L = view_of(d, par);
    const Phys &P = d.P;
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= L.m1 * L.m2) return;
    const int j = t / L.m1, i = t - j * L.m1;
    const int m1 = L.m1, m2 = L.m2, pt = L.pitch, bx = L.bcx, by = L.bcy;
    const double ih = L.inv_h;
    const size_t q = (size_t)j * pt + i;
    const double c0 = L.c[q], mu0 = L.mu[q], p0 = L.p[q], r0 = rho_of(P, c0);
    double uf = 0.0, vf = 0.0;
    if (bx || i > 0) {
        const double cw = ldc(L.c, m1, m2, pt, bx, by, i - 1, j), rw = rho_of(P, cw), Ar = 0.5 * (rw + r0);
        const double st = 0.5 * (r0 * ldc(L.mu, m1, m2, pt, bx, by, i - 1, j) + rw * mu0) * (c0 - cw) * ih;
        uf = L.u[q] + P.dt * frcp(Ar) * (P.inv_M * (st - (p0 - ldc(L.p, m1, m2, pt, bx, by, i - 1, j)) * ih));
    }
    if (by || j > 0) {
        const double cs = ldc(L.c, m1, m2, pt, bx, by, i, j - 1), rs = rho_of(P, cs), Ar = 0.5 * (rs + r0);
        const double st = 0.5 * (r0 * ldc(L.mu, m1, m2, pt, bx, by, i, j - 1) + rs * mu0) * (c0 - cs) * ih;
        vf = L.v[q] + P.dt * frcp(Ar)
                        * (P.inv_M * (st - (p0 - ldc(L.p, m1, m2, pt, bx, by, i, j - 1)) * ih) - P.inv_Fr * (Ar - P.rho_ref));
    }
    d.ub[par ^ 1][q] = uf;
    d.vb[par ^ 1][q] = vf;
}
QN_KERNEL(k_pj_final, __launch_bounds__(BLK), (), ())

// Physical diagnostics of the current state (sec. 8), per-block partials:
//   0: sum c v_cell (v_cell = mean of the cell's south and north faces)
//   1: sum c
//   2: max |div_d u|            3: sum (div_d u)^2          4: sum div_d u
//   5: max height of a c = 1/2 crossing between vertically adjacent cells
//      (linear interpolation; walls in y: interior pairs only)
//   6: min height of such a crossing
//   7: max height of a crossing in the first column (x = h/2)
// (5-7 hold -inf / +inf where there is none.)
#define DIAG_NONE 1e300
template <typename IT> __device__ __forceinline__ void k_diagnostics_body(const IT &it)
{
    __shared__ double sh[BLK / 64][NRED];
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const View L = view_of(d, it_par(it, k));
    const int b = (int)blockIdx.x - it_start(it, k);
    if (b * BLK >= d.m1 * d.m2) return; // pads the list: no partials of its own
    const int t = b * BLK + threadIdx.x;
    double v[NRED] = { 0, 0, 0, 0, 0, -DIAG_NONE, DIAG_NONE, -DIAG_NONE };
    if (t < L.m1 * L.m2) {
        const int j = t / L.m1, i = t - j * L.m1;
        const int m1 = L.m1, m2 = L.m2, pt = L.pitch, bx = L.bcx, by = L.bcy;
        const size_t q = (size_t)j * pt + i;
        const double c = L.c[q];
        const double vs = ldv(L.v, m1, m2, pt, bx, by, i, j), vn = ldv(L.v, m1, m2, pt, bx, by, i, j + 1);
        const double us = ldu(L.u, m1, m2, pt, bx, by, i, j), ue = ldu(L.u, m1, m2, pt, bx, by, i + 1, j);
        v[0] = c * 0.5 * (vs + vn);
        v[1] = c;
        const double dv = (ue - us + vn - vs) * L.inv_h;
        v[2] = fabs(dv);
        v[3] = dv * dv;
        v[4] = dv;
        if (by || j + 1 < m2) {
            const double cn = L.c[(size_t)(j + 1 < m2 ? j + 1 : 0) * pt + i];
            if ((c - 0.5) * (cn - 0.5) < 0.0) {
                const double y = (j + 0.5 + (0.5 - c) / (cn - c)) * d.h;
                v[5] = y;
                v[6] = y;
                if (i == 0) v[7] = y;
            }
        }
    }
    // wave and block reductions: sums for 0, 1, 3, 4; max for 2, 5, 7; min for 6
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int r = 0; r < NRED; r++) {
            const double w = __shfl_xor(v[r], o, 64);
            v[r] = (r == 2 || r == 5 || r == 7) ? fmax(v[r], w) : (r == 6 ? fmin(v[r], w) : v[r] + w);
        }
    }
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0)
#pragma unroll
        for (int r = 0; r < NRED; r++) sh[wv][r] = v[r];
    __syncthreads();
    if (threadIdx.x < NRED) {
        const int r = threadIdx.x;
        double acc = sh[0][r];
        for (int ww = 1; ww < BLK / 64; ww++) {
            const double w = sh[ww][r];
            acc = (r == 2 || r == 5 || r == 7) ? fmax(acc, w) : (r == 6 ? fmin(acc, w) : acc + w);
        }
        d.partials[(size_t)r * part_stride(d) + b] = acc;
    }
}
QN_KERNEL(k_diagnostics, __launch_bounds__(BLK), (), ())

// The reduction of a simulation's partials, in a fixed order: the norms become
// sqrt(h^2 sum r^2), everything goes to device and pinned host memory.
// mode 0: residual reduction (5 norms, sum p, bad count); 1: plain sums;
// 2: the diagnostics slots (sum, max or min per slot as in k_diagnostics).
// Slot q combines by sum (op 0), max (1) or min (2).
__device__ __forceinline__ int red_op(int mode, int q)
{
    return mode != 2 ? 0 : (q == 2 || q == 5 || q == 7) ? 1 : (q == 6 ? 2 : 0);
}
__device__ __forceinline__ double red_comb(int op, double a, double b)
{
    return op == 0 ? a + b : (op == 1 ? fmax(a, b) : fmin(a, b));
}
// slot q of the partials lo, lo + step, .. < hi, by the 16 threads g of the slot
__device__ __forceinline__ double red_slot(const double *p, int mode, int q, int g, int lo, int hi, int step)
{
    const int op = red_op(mode, q);
    double s = op == 0 ? 0.0 : (op == 1 ? -DIAG_NONE : DIAG_NONE);
    for (int b0 = lo + g * step; b0 < hi; b0 += 16 * 16 * step) {
        double v[16]; // loaded before any use
#pragma unroll
        for (int u = 0; u < 16; u++) v[u] = p[min(b0 + u * 16 * step, hi - 1)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 16; u++)
            if (b0 + u * 16 * step < hi) s = red_comb(op, s, v[u]);
    }
    for (int m = 8; m > 0; m >>= 1) s = red_comb(op, s, __shfl_xor(s, m, 64));
    return s;
}
// Many partials are first folded in at most 64 chunks, a workgroup each, the
// chunk's result in its first place: one workgroup reads them at about 35 GB/s
// (16384 partials of 16 slots: 61 us, folded 6.4 + 5.7; 4096: 20 us, folded 5.0 +
// 4.2; 512 with the shift of pbar below: 6.4 us, folded 5.0 + 4.6).
#define FOLD_MIN 512
static __host__ __device__ __forceinline__ int fold_chunk(int n) { return n > FOLD_MIN ? (n + 63) / 64 : 1; }
template <typename IT> __device__ __forceinline__ void k_fold_body(const IT &it, int mode)
{
    static_assert(BLK == 16 * NRED, "16 threads per slot");
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int n = it_cnt(it, k), ch = fold_chunk(n), lo = ((int)blockIdx.x - it_start(it, k)) * ch;
    if (lo >= n) return;
    const int q = threadIdx.x >> 4, g = threadIdx.x & 15;
    double *p = d.partials + (size_t)q * part_stride(d);
    const double s = red_slot(p, mode, q, g, lo, min(lo + ch, n), 1);
    if (g == 0) p[lo] = s; // (the slot's threads, all of this wave, have read the chunk)
}
QN_KERNEL(k_fold, __launch_bounds__(BLK), (int mode), (mode))

// shift (mode 0): also pbar -= mean(pbar), a thread per cell; every workgroup
// sums the pbar partials itself (at most 512, contiguous), which saves the
// launch of a kernel that waits for the sum: 5.4 + 4.1 us became 4.2 on 40 x 40,
// 7.6 + 4.3 became 6.4 on 256 x 512.
template <typename IT> __device__ __forceinline__ void k_finalize_body(const IT &it, int mode, int shift)
{
    __shared__ double sh[BLK / 64];
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int n = it_cnt(it, k), ch = fold_chunk(n), blk = (int)blockIdx.x - it_start(it, k);
    const int st = part_stride(d);
    double psum = 0.0;
    if (shift) {
        const int t = blk * BLK + threadIdx.x, nc = d.m1 * d.m2;
        if (blk * BLK >= nc) return;
        const int j = min(t, nc - 1) / d.m1, i = min(t, nc - 1) - j * d.m1;
        double *const p = d.p + (size_t)j * d.pitch + i;
        const double p0 = *p;
        for (int b = threadIdx.x * ch; b < n; b += BLK * ch) psum += d.partials[(size_t)5 * st + b];
        for (int m = 32; m > 0; m >>= 1) psum += __shfl_xor(psum, m, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = psum;
        __syncthreads();
        psum = sh[0];
#pragma unroll
        for (int w = 1; w < BLK / 64; w++) psum += sh[w];
        if (t < nc) *p = p0 - psum / (double)nc;
    }
    if (blk) return;
    const int q = threadIdx.x >> 4, g = threadIdx.x & 15;
    double x = red_slot(d.partials + (size_t)q * st, mode, q, g, 0, n, ch);
    if (g) return;
    if (mode == 0 && q < 5) x = sqrt(d.h * d.h * x);
    if (shift && q == 5) x = psum;
    d.red[q] = x;
    d.red_host[q] = x;
    // a recorded cycle result: the pbar mean removed from it
    if (mode == 0 && q == 5 && it_acc(it, k) >= 0 && d.amean) d.amean[it_acc(it, k) & 15] = x / (double)(d.m1 * d.m2);
}
QN_KERNEL(k_finalize, __launch_bounds__(BLK), (int mode, int shift), (mode, shift))

// coefficients of the accelerated combination, per item
template <int N> struct AccCoef {
    double g[N][3];
};

// Acceleration step of the cycle iteration: the current iterate w (the last
// cycle result, recorded in ring slot s) becomes w + sum_a g_a (w - w_a), w_a
// the result a + 1 slots back (a < np; its pbar less the mean removed from it,
// which makes it the iterate that result was).  Mixed precision: the next
// correction cycle's right-hand side becomes the same combination of the
// recorded residuals, its linearisation point the combined iterate.
template <typename IT, int N> __device__ __forceinline__ void k_accel_body(const IT &it, const AccCoef<N> &G)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= d.m1 * d.m2 || !d.aw || it_acc(it, k) < 0) return;
    const int j = t / d.m1, i = t - j * d.m1;
    const size_t q = (size_t)j * d.pitch + i, st = (size_t)d.pitch * d.m2;
    const int ac = it_acc(it, k), s = ac & 15, np = ac >> 4, R = d.am, par = it_par(it, k);
    int sl[3];
#pragma unroll
    for (int b = 0; b < 3; b++) sl[b] = (s - 1 - b + R) % R;
    double *const live[5] = { d.c, d.mu, d.p, d.ub[par], d.vb[par] };
    const bool mixed = d.rc != nullptr;
    // every value the cell's combination needs, loaded before any use or
    // store (the stores into the live arrays would otherwise hold back the
    // next field's loads)
    // (global-typed, so that a wait for a scalar load does not also wait for
    // them)
    const double *const aw = d.aw, *const ar = d.ar, *const amean = d.amean;
    double x[5], w[5][3], am[3], xr[5], wr[5][3];
#pragma unroll
    for (int b = 0; b < 3; b++) am[b] = b < np ? lda<1>(amean, sl[b]) : 0.0;
#pragma unroll
    for (int f = 0; f < 5; f++) {
        x[f] = lda<1>(live[f], q);
        xr[f] = mixed ? lda<1>(ar, (size_t)(s * 5 + f) * st + q) : 0.0;
#pragma unroll
        for (int b = 0; b < 3; b++) {
            w[f][b] = b < np ? lda<1>(aw, (size_t)(sl[b] * 5 + f) * st + q) : 0.0;
            wr[f][b] = (mixed && b < np) ? lda<1>(ar, (size_t)(sl[b] * 5 + f) * st + q) : 0.0;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    double y[5];
#pragma unroll
    for (int f = 0; f < 5; f++) {
        double a = x[f];
#pragma unroll
        for (int b = 0; b < 3; b++)
            if (b < np) {
                const double wb = w[f][b] - (f == 2 ? am[b] : 0.0);
                a += G.g[k][b] * (x[f] - wb);
            }
        y[f] = a;
        live[f][q] = a;
    }
    if (mixed) {
        float r[5];
#pragma unroll
        for (int f = 0; f < 5; f++) {
            double a = xr[f];
#pragma unroll
            for (int b = 0; b < 3; b++)
                if (b < np) a += G.g[k][b] * (xr[f] - wr[f][b]);
            r[f] = (float)a;
        }
        d.rc[q] = r[0]; d.rmu[q] = r[1]; d.rp[q] = r[2]; d.ru[q] = r[3]; d.rv[q] = r[4];
        d.xc[q] = (float)y[0]; d.xmu[q] = (float)y[1]; d.xu[q] = (float)y[3]; d.xv[q] = (float)y[4];
    }
}
__global__ __launch_bounds__(BLK) void k_accel(const Desc *d, int w, int cnt, const char *base, unsigned geom, AccCoef<1> G)
{
    k_accel_body(Item1{ d, w, cnt, base, geom }, G);
}
__global__ __launch_bounds__(BLK) void k_accel_n(Items it, AccCoef<MAXITEMS> G) { k_accel_body(it, G); }

// the faces on walls of the level, whose values are zero, in buffer par
__global__ __launch_bounds__(BLK) void k_wall_faces(const Desc *__restrict__ d, int par)
{
    const int t = blockIdx.x * BLK + threadIdx.x;
    if (!d->bcx && t < d->m2) d->ub[par][(size_t)t * d->pitch] = 0.0;
    if (!d->bcy && t < d->m1) d->vb[par][t] = 0.0;
}

// time-n data of the finest level = current iterate; keep mubar, pbar of time n
template <typename IT> __device__ __forceinline__ void k_begin_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= d.m1 * d.m2) return;
    const int j = t / d.m1, i = t - j * d.m1;
    const size_t q = (size_t)j * d.pitch + i;
    const int par = it_par(it, k);
    d.cn[q] = d.c[q];
    d.un[q] = d.ub[par][q];
    d.vn[q] = d.vb[par][q];
    d.mus[q] = d.mu[q];
    d.ps[q] = d.p[q];
    if (d.cnf) {
        d.cnf[q] = (float)d.c[q];
        d.unf[q] = (float)d.ub[par][q];
        d.vnf[q] = (float)d.vb[par][q];
    }
}
QN_KERNEL(k_begin, __launch_bounds__(BLK), (), ())

// time-n data of the coarser level of the item's level
template <typename IT> __device__ __forceinline__ void k_restrict_n_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &F = it_desc(it, k);
    const Desc &C = (&F)[1];
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= C.m1 * C.m2) return;
    const int J = t / C.m1, I = t - J * C.m1;
    const size_t f = (size_t)(2 * J) * F.pitch + 2 * I, q = (size_t)J * C.pitch + I;
    C.cn[q] = 0.25 * (F.cn[f] + F.cn[f + 1] + F.cn[f + F.pitch] + F.cn[f + F.pitch + 1]);
    C.un[q] = 0.5 * (F.un[f] + F.un[f + F.pitch]);
    C.vn[q] = 0.5 * (F.vn[f] + F.vn[f + 1]);
}
QN_KERNEL(k_restrict_n, __launch_bounds__(BLK), (), ())

// restore the state of time n on the finest level (failed step)
template <typename IT> __device__ __forceinline__ void k_restore_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= d.m1 * d.m2) return;
    const int j = t / d.m1, i = t - j * d.m1;
    const size_t q = (size_t)j * d.pitch + i;
    const int par = it_par(it, k);
    d.c[q] = d.cn[q];
    d.ub[par][q] = d.un[q];
    d.vb[par][q] = d.vn[q];
    d.mu[q] = d.mus[q];
    d.p[q] = d.ps[q];
}
QN_KERNEL(k_restore, __launch_bounds__(BLK), (), ())

} // namespace qn
