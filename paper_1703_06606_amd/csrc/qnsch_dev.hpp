// qnsch_dev.hpp -- device side of the FP64 multigrid step (gfx950).
//
// The discrete system is the fully discrete primitive scheme of sec. 6.1
// ((pm-num-mx)-(pm-num-chem), App. A.4-A.6); every equation is written as
// "left side minus right side", N(w) = 0 at time n+1.  The smoother is the
// one of sec. 7.1: per cell a Newton step on the Cahn-Hilliard pair
// (c, mubar), then a Vanka box solve for the four faces and the pressure of
// the cell (or one Newton step on all seven), in red-black order.  The
// projection scheme of sec. 6.2 is the second option (P.scheme, end of file).
//
// Layout: every field of a level is an m2 x pitch array of doubles, row j,
// column i.  Cell fields at cell (i,j); u(i,j) on the west face of cell (i,j)
// (x = i h); v(i,j) on the south face (y = j h).  Ghosts are not stored.
//
// Work is organised in LDS tiles: a workgroup loads a TX x TY block of cells
// with a halo of one cell below and two above in each direction (the reach of
// a Vanka box), applying the boundary conditions of App. A.4 while loading,
// and computes the cell functions of the time-n data (rho^n, mu(c^n), m(c^n))
// and rho(c) once per tile element.  The equations below then read the tile
// without any boundary logic.
#pragma once
#include <hip/hip_runtime.h>

namespace qn {

struct Phys {
    double rho1, rho2, rho12, drho;  // rho(c) = rho12 / (drho c + rho1)
    double visc1, visc2, visc12, dvisc;
    double alpha, inv_Re, inv_M, inv_Pe, K1, K2, K3, inv_Fr, rho_ref, mob_reg;
    double inv_dt, dt;
    int coupled; // smoother: 1 = one Newton step on the seven-unknown box, 0 = the two steps
    int scheme;  // 0 = primitive scheme (sec. 6.1), 1 = projection scheme (sec. 6.2)
};

// Coefficients of the equations on one level for one step size, products of
// the physical constants and powers of h that every cell would otherwise form
// again (there is no scalar FP64 arithmetic: a product of two uniform values
// costs each wave a vector instruction).  R: double, or float for the
// correction smoother.
template <typename R> struct Kon {
    R ih, hih;         // 1/h, 1/(2h)
    R idt, hidt;       // 1/dt, 1/(2dt)
    R ka;              // 1/(16 h): advection of a momentum row
    R kv, kv34;        // 1/(3 Re h^2) and 3/4 of it: viscous terms
    R kp, hkp, iM;     // 1/(M h) and half of it: pressure, surface tension; 1/M
    R km, akm;         // 1/(2 Pe h^2), alpha times it: mobility fluxes
    R alpha;
    R K1, kg, kl;      // bulk terms; K2/(4 h^2); K3/(8 h^2)
    R inv_Fr, rho_ref; // gravity on the north-south faces
    R dt2;             // 2 dt (projection equation)
};

struct View {
    double *c, *mu, *p;         // cell unknowns
    const double *u, *v;        // face unknowns (the buffer being read)
    const double *cn, *un, *vn; // time-n data
    int m1, m2, pitch;
    int bcx, bcy;               // 0 wall, 1 periodic
    double inv_h;
};

struct Rhs {
    const double *fc, *fmu, *fp, *fu, *fv; // FAS right-hand side; NULL = 0
};

// loads and stores through a pointer of address space AS (1: global memory,
// 3: LDS, 0: either).  A level's arrays reach the kernels inside structures,
// so without it the compiler issues generic accesses, which count as LDS
// accesses too: every wait for an LDS read would then also wait for the
// outstanding global loads.
template <int AS, typename R> __device__ __forceinline__ R lda(const R *p, size_t k)
{
    if constexpr (AS == 1)
        return ((const __attribute__((address_space(1))) R *)p)[k];
    else if constexpr (AS == 3)
        return ((const __attribute__((address_space(3))) R *)p)[k];
    else
        return p[k];
}
template <int AS, typename R> __device__ __forceinline__ void sta(R *p, size_t k, R v)
{
    if constexpr (AS == 1)
        ((__attribute__((address_space(1))) R *)p)[k] = v;
    else if constexpr (AS == 3)
        ((__attribute__((address_space(3))) R *)p)[k] = v;
    else
        p[k] = v;
}

// --------------------------------------------------------------------------
// loaders with boundary conditions (used only by the tile loader)

__device__ __forceinline__ int wrapi(int k, int n) { return k < 0 ? k + n : (k >= n ? k - n : k); }

// cell field: Neumann mirror or periodic image (x first, then y)
template <typename R>
__device__ __forceinline__ R ldc(const R *f, int m1, int m2, int pitch, int bcx, int bcy, int i, int j)
{
    if (i < 0 || i >= m1) i = bcx ? wrapi(i, m1) : (i < 0 ? 0 : m1 - 1);
    if (j < 0 || j >= m2) j = bcy ? wrapi(j, m2) : (j < 0 ? 0 : m2 - 1);
    return f[(size_t)j * pitch + i];
}
// east-west face field at x = i h, row j: zero on (and beyond) x-walls,
// reflected (ghost = -interior) across y-walls
template <typename R>
__device__ __forceinline__ R ldu(const R *f, int m1, int m2, int pitch, int bcx, int bcy, int i, int j)
{
    if (bcx) i = wrapi(i, m1);
    else if (i <= 0 || i >= m1) return R(0);
    if (j < 0 || j >= m2) {
        if (bcy) j = wrapi(j, m2);
        else return -f[(size_t)(j < 0 ? 0 : m2 - 1) * pitch + i];
    }
    return f[(size_t)j * pitch + i];
}
template <typename R>
__device__ __forceinline__ R ldv(const R *f, int m1, int m2, int pitch, int bcx, int bcy, int i, int j)
{
    if (bcy) j = wrapi(j, m2);
    else if (j <= 0 || j >= m2) return R(0);
    if (i < 0 || i >= m1) {
        if (bcx) i = wrapi(i, m1);
        else return -f[(size_t)j * pitch + (i < 0 ? 0 : m1 - 1)];
    }
    return f[(size_t)j * pitch + i];
}
// Where a tile element (i, j) comes from, for each kind of field: the array
// index and a sign (1; -1 for a reflected tangential ghost of a face field;
// 0 for a wall face, which is zero) as ldc, ldu, ldv resolve them; beyond the
// reach of any cell of the level (a tile larger than the level) every sign
// is 0 and the element is all zero.  Computing all sources first lets a
// thread issue all its loads at once.
struct TileSrc {
    int c, u, v;    // array indices (always valid)
    int sc, su, sv; // signs
};
__device__ __forceinline__ TileSrc tile_src(int m1, int m2, int pitch, int bcx, int bcy, int i, int j)
{
    TileSrc s;
    if (i > m1 + 1 || j > m2 + 1) {
        s.c = s.u = s.v = 0;
        s.sc = s.su = s.sv = 0;
        return s;
    }
    int ic = i, jc = j;
    if (ic < 0 || ic >= m1) ic = bcx ? wrapi(ic, m1) : (ic < 0 ? 0 : m1 - 1);
    if (jc < 0 || jc >= m2) jc = bcy ? wrapi(jc, m2) : (jc < 0 ? 0 : m2 - 1);
    s.c = jc * pitch + ic;
    s.sc = 1;
    int iu = i, ju = j;
    s.su = 1;
    if (bcx) iu = wrapi(iu, m1);
    else if (iu <= 0 || iu >= m1) { s.su = 0; iu = 0; }
    if (ju < 0 || ju >= m2) {
        if (bcy) ju = wrapi(ju, m2);
        else { s.su = -s.su; ju = ju < 0 ? 0 : m2 - 1; }
    }
    s.u = ju * pitch + iu;
    int iv = i, jv = j;
    s.sv = 1;
    if (bcy) jv = wrapi(jv, m2);
    else if (jv <= 0 || jv >= m2) { s.sv = 0; jv = 0; }
    if (iv < 0 || iv >= m1) {
        if (bcx) iv = wrapi(iv, m1);
        else { s.sv = -s.sv; iv = iv < 0 ? 0 : m1 - 1; }
    }
    s.v = jv * pitch + iv;
    return s;
}
// the sources of tile_src as level coordinates: cell (ic, jc), u face
// (iu, ju), v face (iv, jv), resolved by the same rules (tile_src keeps its own
// copy: composing it from this one measured slower in the tile loads)
struct TileSrcIJ {
    int ic, jc, iu, ju, iv, jv;
    int sc, su, sv;
};
__device__ __forceinline__ TileSrcIJ tile_src_ij(int m1, int m2, int bcx, int bcy, int i, int j)
{
    TileSrcIJ s;
    if (i > m1 + 1 || j > m2 + 1) {
        s.ic = s.jc = s.iu = s.ju = s.iv = s.jv = 0;
        s.sc = s.su = s.sv = 0;
        return s;
    }
    int ic = i, jc = j;
    if (ic < 0 || ic >= m1) ic = bcx ? wrapi(ic, m1) : (ic < 0 ? 0 : m1 - 1);
    if (jc < 0 || jc >= m2) jc = bcy ? wrapi(jc, m2) : (jc < 0 ? 0 : m2 - 1);
    s.ic = ic; s.jc = jc;
    s.sc = 1;
    int iu = i, ju = j;
    s.su = 1;
    if (bcx) iu = wrapi(iu, m1);
    else if (iu <= 0 || iu >= m1) { s.su = 0; iu = 0; }
    if (ju < 0 || ju >= m2) {
        if (bcy) ju = wrapi(ju, m2);
        else { s.su = -s.su; ju = ju < 0 ? 0 : m2 - 1; }
    }
    s.iu = iu; s.ju = ju;
    int iv = i, jv = j;
    s.sv = 1;
    if (bcy) jv = wrapi(jv, m2);
    else if (jv <= 0 || jv >= m2) { s.sv = 0; jv = 0; }
    if (iv < 0 || iv >= m1) {
        if (bcx) iv = wrapi(iv, m1);
        else { s.sv = -s.sv; iv = iv < 0 ? 0 : m1 - 1; }
    }
    s.iv = iv; s.jv = jv;
    return s;
}
template <typename R> __device__ __forceinline__ R signed_val(int sg, R x) { return sg > 0 ? x : (sg < 0 ? -x : R(0)); }

__device__ __forceinline__ bool u_unk(const View &L, int i) { return L.bcx || (i >= 1 && i <= L.m1 - 1); }
__device__ __forceinline__ bool v_unk(const View &L, int j) { return L.bcy || (j >= 1 && j <= L.m2 - 1); }

// --------------------------------------------------------------------------
// material laws (sec. 2.1, sec. 6.1)

// reciprocal: hardware estimate refined by two Newton steps (relative error a
// few ulp, far below the solver tolerances)
__device__ __forceinline__ double frcp(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}
__device__ __forceinline__ double rho_of(const Phys &P, double c) { return P.rho12 * frcp(P.drho * c + P.rho1); }
__device__ __forceinline__ double visc_of(const Phys &P, double c) { return P.visc12 * frcp(P.dvisc * c + P.visc1); }
__device__ __forceinline__ double mob_of(const Phys &P, double c)
{
    double q = c * (1.0 - c);
    return sqrt(q * q + P.mob_reg);
}
__device__ __forceinline__ double dwell(double c)
{
    double q = c * (c - 1.0);
    return 0.25 * q * q;
}

// --------------------------------------------------------------------------
// LDS tile

// fields of a tile element, kept together (T_U2, T_V2: the new faces of a
// sweep that stays in the tile).  A cell's neighbours are then a few base
// addresses with constant offsets, and adjacent fields load together as 16
// bytes; with one array per field every access of a relaxation needed an
// address of its own.  The element of 14 doubles spreads the cells of a
// colour (every second element) over half of the LDS banks.
enum { T_C = 0, T_CN, T_MU, T_P, T_RN, T_MV, T_RS, T_MOB, T_U, T_UN, T_V, T_VN, T_NF, T_U2 = T_NF, T_V2, T_ES };
// the correction smoother's further fields (its T_MU, T_P, T_U, T_V hold
// corrections): the correction of c and the change of density it induces
enum { L_DC = T_ES, L_DRS, L_ES = 20 };

// A tile covers level cells i0-1 .. i0+W-2, j0-1 .. j0+H-2 (a tile of TX
// columns: W = TX+3) in rows of S elements; at(i, j), q(f, i, j) take level
// coordinates.  S is even: the cells of one colour are every second element,
// from another start in every other row, and with an even S the rows of odd
// start then use the LDS banks that the others leave free.
template <typename R, int ES_> struct TileT {
    static constexpr int ES = ES_;
    R *s; // W*H elements of ES values in LDS
    int i0, j0, W, H, S;
    __device__ __forceinline__ int idx(int i, int j) const { return (j - j0 + 1) * S + (i - i0 + 1); }
    __device__ __forceinline__ R *at(int i, int j) const { return s + idx(i, j) * ES; }
    __device__ __forceinline__ R q(int f, int i, int j) const { return at(i, j)[f]; }
};
typedef TileT<double, T_ES> Tile;
// without the second face slot: the residual kernels (a half-sweep's lanes, on
// every second element, meet fewer banks at 12 values: 41.1 us against 37.9 at 14)
typedef TileT<double, T_NF> Tile1;

// the element n elements from s (a row is S of them).  The offset is a
// multiple of the element's size in the code, too: the compiler then knows the
// element to be aligned to 16 bytes and loads a pair of fields as one
// ds_read_b128; otherwise it makes a ds_read2_b64 of it, which takes the LDS
// 15.5 cycles per wave instead of 4.5 (MI355X).
template <int ES, typename R> __device__ __forceinline__ R *el(R *s, int n) { return s + n * ES; }

// an element's fields from its eight loaded values (c, mubar, pbar, u, v, c^n,
// u^n, v^n) and the signs of its faces
__device__ __forceinline__ void tile_put(const Phys &P, double *t, int su, int sv, const double (&v)[8])
{
    t[T_C] = v[0];
    t[T_CN] = v[5];
    t[T_MU] = v[1];
    t[T_P] = v[2];
    t[T_RN] = rho_of(P, v[5]);
    t[T_MV] = visc_of(P, v[5]);
    t[T_RS] = rho_of(P, v[0]);
    t[T_MOB] = mob_of(P, v[5]);
    t[T_U] = signed_val(su, v[3]);
    t[T_UN] = signed_val(su, v[6]);
    t[T_V] = signed_val(sv, v[4]);
    t[T_VN] = signed_val(sv, v[7]);
}
template <typename TT> __device__ __forceinline__ void tile_zero(const TT &T, int e)
{
#pragma unroll
    for (int f = 0; f < TT::ES; f++) T.s[e * TT::ES + f] = 0;
}

// true if every element of the tile (halo included) is an interior element
// of the level for every field, so that no boundary image is involved: cells
// and faces 1 .. m-1 in each direction
__device__ __forceinline__ bool tile_inner(int m1, int m2, int i0, int j0, int W, int H)
{
    return i0 >= 2 && j0 >= 2 && i0 + W - 2 <= m1 - 1 && j0 + H - 2 <= m2 - 1;
}

// cooperative load of a tile of a level in global memory (all threads of the
// block take part; the caller synchronises afterwards).  NE elements per
// thread are loaded together: their sources first, then every load, then the
// signs and cell functions (an element past the end is clamped to a valid
// one and not stored).
// (D: the level's descriptor, whose constants are read behind the loads)
template <int NE, int NT, typename TT, typename D> __device__ __forceinline__ void tile_load(const D &d, const View &L, const TT &T)
{
    const int n = T.W * T.H;
    double v[NE][8];
    if (tile_inner(L.m1, L.m2, T.i0, T.j0, T.W, T.H)) {
#pragma unroll
        for (int k = 0; k < NE; k++) {
            const int e = min((int)threadIdx.x + k * NT, n - 1), b = e / T.W, a = e - b * T.W;
            const size_t q = (size_t)((T.j0 - 1 + b) * L.pitch + (T.i0 - 1 + a));
            const double *src[8] = { L.c, L.mu, L.p, L.u, L.v, L.cn, L.un, L.vn };
#pragma unroll
            for (int f = 0; f < 8; f++) v[k][f] = lda<1>(src[f], q);
        }
        __builtin_amdgcn_sched_barrier(0);
        const Phys P = d.P;
#pragma unroll
        for (int k = 0; k < NE; k++) {
            const int e = threadIdx.x + k * NT, b = e / T.W, a = e - b * T.W;
            if (e < n) tile_put(P, T.s + (b * T.S + a) * TT::ES, 1, 1, v[k]);
        }
        return;
    }
    TileSrc s[NE];
#pragma unroll
    for (int k = 0; k < NE; k++) {
        const int e = min((int)threadIdx.x + k * NT, n - 1), b = e / T.W, a = e - b * T.W;
        s[k] = tile_src(L.m1, L.m2, L.pitch, L.bcx, L.bcy, T.i0 - 1 + a, T.j0 - 1 + b);
        const double w[8] = { lda<1>(L.c, s[k].c), lda<1>(L.mu, s[k].c), lda<1>(L.p, s[k].c), lda<1>(L.u, s[k].u),
                              lda<1>(L.v, s[k].v), lda<1>(L.cn, s[k].c), lda<1>(L.un, s[k].u), lda<1>(L.vn, s[k].v) };
#pragma unroll
        for (int f = 0; f < 8; f++) v[k][f] = w[f];
    }
    __builtin_amdgcn_sched_barrier(0);
    const Phys P = d.P;
#pragma unroll
    for (int k = 0; k < NE; k++) {
        const int e = threadIdx.x + k * NT, b = e / T.W, a = e - b * T.W;
        if (e >= n) continue;
        if (s[k].sc == 0) tile_zero(T, b * T.S + a);
        else tile_put(P, T.s + (b * T.S + a) * TT::ES, s[k].su, s[k].sv, v[k]);
    }
}

// Images of a level that is resident in its tile: the elements outside
// the level, [-1, m+1] on each axis without [0, m-1], in the order the ring is
// walked; for each its element and those of its sources (a cell, a u face, a v
// face of the level) with the signs of the faces, as tile_src_ij gives them.
struct alignas(16) Image {
    int e, c, u, v; // element; elements of the sources, faces' signs + 1 in the low two bits
};
__host__ __device__ __forceinline__ int ring_size(int m1, int m2) { return (m1 + 3) * (m2 + 3) - m1 * m2; }
// entry k of the ring
template <typename TT> __device__ __forceinline__ Image ring_entry(const TT &T, int m1, int m2, int bcx, int bcy, int k)
{
    int i, j;
    // rows -1, m2, m2 + 1, then columns -1, m1, m1 + 1 of the other rows
    if (k < 3 * (m1 + 3)) {
        const int r = k / (m1 + 3);
        i = k - r * (m1 + 3) - 1;
        j = r == 0 ? -1 : m2 + r - 1;
    } else {
        const int q = k - 3 * (m1 + 3), r = q / 3, s = q - 3 * r;
        j = r;
        i = s == 0 ? -1 : m1 + s - 1;
    }
    const TileSrcIJ q = tile_src_ij(m1, m2, bcx, bcy, i, j);
    Image g;
    g.e = T.idx(i, j);
    g.c = T.idx(q.ic, q.jc);
    g.u = T.idx(q.iu, q.ju) * 4 + q.su + 1;
    g.v = T.idx(q.iv, q.jv) * 4 + q.sv + 1;
    return g;
}

// --------------------------------------------------------------------------
// The equations of a cell come in two parts, one per axis, of the same form on
// transposed strides.  A relaxation takes a pair of adjacent lanes per cell:
// lane 0 the x part, lane 1 the y part, the partial sums exchanged between
// them (one instruction stream, the shorter chain); or one lane that takes
// both parts in turn (fewer instructions per cell).  A residual takes one
// lane per cell.  Multiply-adds are contracted within an expression only
// (-ffp-contract=on), so every kernel that shares these functions computes
// the same values.

// (ES: values per element)
template <int ES> struct Ax {
    int dn, dt;          // elements to the next one along the normal / tangential axis
    int fn, ft, fo;      // own velocity (T_U or T_V, or T_U2, T_V2), other velocity, new own velocity
    int fnn, ftn;        // own and other velocity of time n
    bool per, pert;      // periodic along the axis / the other one
    int ia, ma, it, mt;  // cell index and count along the axis / the other one
    int hlf;             // 0 x, 1 y
};

// slot: the faces are in T_U, T_V and a sweep that stays in the tile puts the
// new ones into T_U2, T_V2 (0), or the other way round (1)
template <typename V, typename TT>
__device__ __forceinline__ Ax<TT::ES> make_ax(const V &L, const TT &T, int i, int j, int hlf, int slot = 0)
{
    Ax<TT::ES> a;
    a.hlf = hlf;
    a.dn = hlf ? T.S : 1;
    a.dt = hlf ? 1 : T.S;
    a.fn = slot ? T_U2 + hlf : T_U + 2 * hlf;
    a.ft = slot ? T_V2 - hlf : T_V - 2 * hlf;
    a.fo = slot ? T_U + 2 * hlf : T_U2 + hlf;
    a.fnn = T_UN + 2 * hlf;
    a.ftn = T_VN - 2 * hlf;
    a.per = hlf ? L.bcy : L.bcx;
    a.pert = hlf ? L.bcx : L.bcy;
    a.ia = hlf ? j : i;
    a.ma = hlf ? L.m2 : L.m1;
    a.it = hlf ? i : j;
    a.mt = hlf ? L.m1 : L.m2;
    return a;
}

// value of the partner lane (lane ^ 1): a DPP quad permutation [1,0,3,2]
// within the wave's registers, no LDS round trip
__device__ __forceinline__ int other(int x) { return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false); }
__device__ __forceinline__ float other(float x) { return __int_as_float(other(__float_as_int(x))); }
__device__ __forceinline__ double other(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = other((int)(b & 0xffffffffll)), hi = other((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The axis part of the cell equations at element s, in the combinations that
// the equations take them in:
//   s1  advection of c (App. A.5) - (1/Pe) L_m(mubar + alpha pbar)   (phase)
//   s2  divergence - (alpha/Pe) L_m(mubar + alpha pbar)              (mass)
//   sm  (1/Pe) times the sum of the mobilities over h^2 (minus the diagonal of
//       (1/Pe) L_m)
//   g   4 h^2 times the average of |grad c|^2 over the two time levels
//   lr  8 h^2 times the capillary divergence (App. A.6)
//   j   what g and lr add to d(chemical row)/dc besides the pointwise terms
// (r, drs: -alpha rho rho^n and rho'(c) of the cell).  A face on a wall
// carries no flux: the mirrored ghost equals the cell, so every difference
// across it is zero; the masks wP, wM matter for derivatives only.
template <typename R> struct CellSum {
    R s1, s2, sm, g, lr, j;
};
// u0, uP: the velocity on the cell's low and high face along the axis.  PJ:
// the projection scheme, whose advection takes c and rho of time n+1.
template <bool PJ, int ES>
__device__ __forceinline__ CellSum<double> axis_cell(const Kon<double> &K, const double *s, const Ax<ES> &a, double r,
                                                     double drs, double u0, double uP)
{
    const bool wP = a.per || a.ia < a.ma - 1, wM = a.per || a.ia > 0;
    const double *sP = el<ES>(s, a.dn), *sM = el<ES>(s, -a.dn);
    const double mP = sP[T_MOB] + s[T_MOB], mM = sM[T_MOB] + s[T_MOB];
    const double S = s[T_MU] + K.alpha * s[T_P];
    const double fP = (sP[T_MU] + K.alpha * sP[T_P]) - S, fM = S - (sM[T_MU] + K.alpha * sM[T_P]);
    const double flux = mP * fP - mM * fM;
    const double gP = sP[T_CN] - s[T_CN], gM = s[T_CN] - sM[T_CN], dP = sP[T_C] - s[T_C], dM = s[T_C] - sM[T_C];
    CellSum<double> x;
    const double aP = PJ ? sP[T_RS] * dP : sP[T_RN] * gP, aM = PJ ? sM[T_RS] * dM : sM[T_RN] * gM;
    const double adv = aP * uP + aM * u0;
    x.s1 = K.hih * adv - K.km * flux;
    x.s2 = K.ih * (uP - u0) - K.akm * flux;
    x.sm = K.km * ((wP ? mP : 0.0) + (wM ? mM : 0.0));
    x.g = (dP * dP + dM * dM) + (gP * gP + gM * gM);
    const double hP = dP + gP, hM = dM + gM;
    const double R0 = s[T_RS] + s[T_RN];
    const double RP = (sP[T_RS] + sP[T_RN]) + R0, RM = (sM[T_RS] + sM[T_RN]) + R0;
    x.lr = RP * hP - RM * hM;
    const double w = (wP ? RP : 0.0) + (wM ? RM : 0.0);
    x.j = K.kl * (drs * (hP - hM) - w) - (2.0 * K.kg * r) * (dM - dP);
    return x;
}
template <typename R> __device__ __forceinline__ CellSum<R> other(const CellSum<R> &x)
{
    return { other(x.s1), other(x.s2), other(x.sm), other(x.g), other(x.lr), other(x.j) };
}
template <typename R> __device__ __forceinline__ CellSum<R> operator+(const CellSum<R> &x, const CellSum<R> &y)
{
    return { x.s1 + y.s1, x.s2 + y.s2, x.sm + y.sm, x.g + y.g, x.lr + y.lr, x.j + y.j };
}

// cell equations: phase (pm-num-phase), chemical potential (pm-num-chem) and
// mass (pm-num-mass), with the Jacobian entries the smoother needs, from the
// sum of the axis parts
struct CellEq {
    double Nc, Nmu, Np;
    double Jcc, Jcm, Jmc, Jmm; // d(Nc,Nmu)/d(c,mu) at the cell
};

// pointwise quantities of the cell that the axis parts need
__device__ __forceinline__ void cell_r(const Kon<double> &K, const double *s, double &r, double &drs)
{
    const double t = -K.alpha * s[T_RS];
    r = t * s[T_RN];
    drs = t * s[T_RS];
}
__device__ __forceinline__ CellEq cell_eq(const Kon<double> &K, const double *s, const CellSum<double> &x, double r,
                                          double drs)
{
    const double c = s[T_C], n = s[T_CN], mu = s[T_MU], rs = s[T_RS], rn = s[T_RN];
    CellEq q;
    q.Nc = K.idt * (rs * (c - n)) + x.s1;
    q.Np = x.s2;
    // time averages of sec. 4.1; pointwise |grad_D c|^2 = a_x((D_x c)^2) + a_y((D_y c)^2)
    const double rh = 0.5 * (rs + rn);
    const double q1 = c * (c - 1.0), q0 = n * (n - 1.0), t = c + n - 1.0, qs = q1 + q0;
    const double g = 0.25 * qs * t;
    const double Fh = 0.125 * (q1 * q1 + q0 * q0);
    const double G = K.kg * x.g + K.K1 * Fh; // K2 |grad c|^2 + K1 F, both times r
    q.Nmu = rs * mu - K.K1 * (rh * g) - G * r + K.kl * x.lr;
    // Jacobian in (c_ij, mubar_ij); rho' = -alpha rho^2
    q.Jcc = K.idt * (drs * (c - n) + rs);
    q.Jcm = x.sm;
    q.Jmm = rs;
    const double dg = 0.25 * ((2.0 * c - 1.0) * t + qs);
    const double f1 = q1 * (c - 0.5);   // F'(c)
    const double dr = -K.alpha * rs * r; // dr/dc
    q.Jmc = drs * mu - K.K1 * (0.5 * (drs * g + f1 * r) + rh * dg) - G * dr + x.j;
    return q;
}

// --------------------------------------------------------------------------
// momentum equation (pm-num-mx) on the face stored at element s (the west
// face of its cell on the x axis, the south face on the y axis), with the
// derivative with respect to the face's own velocity.  Advection (e1e1-1) plus
// the half-divergence term (e1e1-2) are used in their skew form
//   1/(2h) [w_R u_{+1} - w_L u_{-1} + Z_t u_{t+1} - Z_b u_{t-1}],
// which is the same sum with the terms on the face's own value cancelled.
// (it = tangential index of the face's row.)  PJ: the projection scheme's
// intermediate velocity (pj-num-mx), which has neither pressure, surface
// tension nor gravity (they act in (pj-num-pjx)).  The two faces of a box
// share their common terms (the compiler finds them: the expressions are the
// same).
template <typename R> struct FaceEq {
    R N, diag;
};

// LIN: the equation's linearisation at w^ applied to a correction (the
// correction smoother): uh is the face's velocity at w^, which multiplies the
// change of the density average (field L_DRS); gravity and u^n drop out.
template <typename R, bool PJ, bool LIN, int ES>
__device__ __forceinline__ FaceEq<R> face_eq(const Kon<R> &K, const R *s, const Ax<ES> &a, R uh = R(0))
{
    const int dn = a.dn, dt = a.dt, fn = a.fn, ft = a.ft, fnn = a.fnn, ftn = a.ftn;
    const R *L = el<ES>(s, -dn), *Rn = el<ES>(s, dn), *Lt = el<ES>(L, dt), *Lb = el<ES>(L, -dt), *St = el<ES>(s, dt), *Sb = el<ES>(s, -dt);
    const R rL = L[T_RN], rR = s[T_RN], mL = L[T_MV], mR = s[T_MV];
    const R a1 = rL + rR, b1 = mL + mR;
    const R At = (Lt[T_RN] + St[T_RN]) + a1, Ab = (Lb[T_RN] + Sb[T_RN]) + a1;
    const R mt = (Lt[T_MV] + St[T_MV]) + b1, mb = (Lb[T_MV] + Sb[T_MV]) + b1;
    const R hA = R(0.5) * ((L[T_RS] + s[T_RS]) - a1);
    const R un0 = s[fnn];
    const R wL = rL * (L[fnn] + un0), wR = rR * (un0 + Rn[fnn]);
    const R Ct = At * (Lt[ftn] + St[ftn]), Cb = Ab * (L[ftn] + s[ftn]);
    const R u0 = s[fn], uE = Rn[fn], uW = L[fn], uN = St[fn], uS = Sb[fn];
    // (4 d_n u + d_t v) h of the cells on both sides
    const R thR = R(4) * (uE - u0) + (St[ft] - s[ft]), thL = R(4) * (u0 - uW) + (Lt[ft] - L[ft]);
    const R advn = wR * uE - wL * uW;
    const R adv = R(4) * advn + (Ct * uN - Cb * uS);
    const R v1 = mR * thR - mL * thL, v2 = mt * (uN - u0) - mb * (u0 - uS);
    FaceEq<R> q;
    R td = a1 * (LIN ? u0 : u0 - un0) + hA * u0; // time derivative
    if (LIN) td = td + R(0.5) * (L[L_DRS] + s[L_DRS]) * uh;
    q.N = K.hidt * td + K.ka * adv - (K.kv * v1 + K.kv34 * v2);
    if (!PJ) {
        const R sf = (rR * L[T_MU] + rL * s[T_MU]) * (s[T_CN] - L[T_CN]);
        q.N += K.kp * (s[T_P] - L[T_P]) - K.hkp * sf;
        if (!LIN && a.hlf) q.N += K.inv_Fr * (R(0.5) * a1 - K.rho_ref);
    }
    // own-face derivative; across a tangential wall the reflected ghost doubles
    // the viscous coupling and the advection coefficient enters with a sign flip
    q.diag = K.hidt * (a1 + hA) + R(4) * (K.kv * b1) + K.kv34 * (mt + mb);
    if (!a.pert) {
        if (a.it == a.mt - 1) q.diag += K.kv34 * mt - K.ka * Ct;
        if (a.it == 0) q.diag += K.kv34 * mb + K.ka * Cb;
    }
    return q;
}

// --------------------------------------------------------------------------
// The box of a cell.  Along an axis its two faces satisfy
//   V x = b + s t - q dc,   V = (dlo, alh; ahl, dhi),  s = (1, -1),
//   t = gd D_o - gp p,
// with D = x_hi - x_lo and D_o that of the other axis: the viscous coupling of
// the axes and the pressure enter an axis through t alone, the cell's c and
// mubar (coupled box; mubar eliminated by the chemical row as kbm - kmc dc)
// through q and b.  The mass row takes the D of both axes, the phase row a.x
// of both (a: the advection weights of App. A.5).  So each axis inverts its
// own 2x2 block for the three right-hand sides, and the rest is a system in
// (D_x, D_y), then (p, dc).  (A face on a wall is no unknown: identity row,
// zero right-hand sides.)
template <typename R> struct BoxAx {
    R xb[2], xs[2], xq[2]; // V^-1 b, V^-1 s, V^-1 q: low and high face
    R Db, Ds, Dq;          // their D
    R Ab, As, Aq;          // their a.x
};
__device__ __forceinline__ double frcp_(double x) { return frcp(x); }
__device__ __forceinline__ float frcp_(float x) { return __builtin_amdgcn_rcpf(x); }

template <typename R>
__device__ __forceinline__ BoxAx<R> box_axis(R dlo, R dhi, R alh, R ahl, R blo, R bhi, R slo, R shi, R qlo, R qhi,
                                             R alo, R ahi)
{
    const R id = frcp_(dlo * dhi - alh * ahl);
    const R v00 = dhi * id, v01 = -(alh * id), v10 = -(ahl * id), v11 = dlo * id;
    BoxAx<R> x;
    x.xb[0] = v00 * blo + v01 * bhi;
    x.xb[1] = v10 * blo + v11 * bhi;
    x.xs[0] = v00 * slo + v01 * shi;
    x.xs[1] = v10 * slo + v11 * shi;
    x.xq[0] = v00 * qlo + v01 * qhi;
    x.xq[1] = v10 * qlo + v11 * qhi;
    x.Db = x.xb[1] - x.xb[0];
    x.Ds = x.xs[1] - x.xs[0];
    x.Dq = x.xq[1] - x.xq[0];
    x.Ab = alo * x.xb[0] + ahi * x.xb[1];
    x.As = alo * x.xs[0] + ahi * x.xs[1];
    x.Aq = alo * x.xq[0] + ahi * x.xq[1];
    return x;
}
// the parts of the other axis that box_solve needs
template <typename R> struct BoxOther {
    R Db, Ds, Dq, Ab, As, Aq;
};
template <typename R> __device__ __forceinline__ BoxOther<R> box_other(const BoxAx<R> &x)
{
    return { other(x.Db), other(x.Ds), other(x.Dq), other(x.Ab), other(x.As), other(x.Aq) };
}
// p, dc and t of both axes (to: own, tt: other) from
//   mass row:   ih (D_x + D_y) + Jpp p + Jcp (kbm - kmc dc) = bp
//   phase row:  a.x + a.y + Jcp p + Jc dc = r1,  Jc = Jcc - Jcm kmc (r1 less Jcm kbm)
// cpl = false: the Vanka box alone (dc = 0)
template <typename R>
__device__ __forceinline__ void box_solve(const BoxAx<R> &x, const BoxOther<R> &y, bool cpl, R gd, R gp, R ih, R Jpp,
                                          R Jcp, R kmc, R kbm, R Jc, R bp, R r1, R &p, R &dc, R &to, R &tt)
{
    // (D_x, D_y) = D0 + Dp p + Dc dc
    const R gx = gd * x.Ds, gy = gd * y.Ds;
    const R idl = frcp_(R(1) - gx * gy);
    const R X0 = (x.Db + gx * y.Db) * idl, Y0 = (y.Db + gy * x.Db) * idl;
    const R gpi = -gp * idl;
    const R Xp = (x.Ds + gx * y.Ds) * gpi, Yp = (y.Ds + gy * x.Ds) * gpi;
    const R Mp = ih * (Xp + Yp) + Jpp;
    if (!cpl) {
        p = (bp - ih * (X0 + Y0)) * frcp_(Mp);
        dc = R(0);
        to = gd * (Y0 + Yp * p) - gp * p;
        tt = gd * (X0 + Xp * p) - gp * p;
        return;
    }
    const R Xc = -(x.Dq + gx * y.Dq) * idl, Yc = -(y.Dq + gy * x.Dq) * idl;
    const R Mc = ih * (Xc + Yc) - Jcp * kmc, M0 = (bp - Jcp * kbm) - ih * (X0 + Y0);
    const R tp = gd * Yp - gp, sp = gd * Xp - gp;
    const R Pp = (Jcp + x.As * tp) + y.As * sp;
    const R Pc = (Jc - (x.Aq + y.Aq)) + gd * (x.As * Yc + y.As * Xc);
    const R P0 = (r1 - (x.Ab + y.Ab)) - gd * (x.As * Y0 + y.As * X0);
    const R idt = frcp_(Mp * Pc - Mc * Pp);
    p = (M0 * Pc - Mc * P0) * idt;
    dc = (Mp * P0 - Pp * M0) * idt;
    to = gd * (Y0 + Yc * dc) + tp * p;
    tt = gd * (X0 + Xc * dc) + sp * p;
}

// face right-hand side of the lane's axis: the select is taken on the pointer
// values (a select between the two struct members made the compiler stage
// them in scratch memory)
__device__ __forceinline__ const double *face_rhs(const Rhs &F, int hlf)
{
    const uintptr_t a = (uintptr_t)F.fu, b = (uintptr_t)F.fv;
    return (const double *)(hlf ? b : a);
}

// --------------------------------------------------------------------------
// The neighbourhood of a cell that a lane's part of its relaxation reads,
// copied into registers: elements n = -1 .. 2 along the lane's axis, t = -1 ..
// 1 across it, at h[((n + 1) * 3 + t + 1) * ES], with the velocities in the
// lane's order (own: T_U, T_UN).  All loads are issued before anything uses
// one.  Where a launch lasts as long as the chain of its relaxations (few
// waves, registers to spare), reading the tile at each use instead waits for
// LDS some twenty times per relaxation: it cost 8 of 65 us for 24 half-sweeps in
// one workgroup.
// A neighbour across a wall is read at its source in the level (the cell next
// to the wall; the own velocity past a wall along the axis' side changes sign),
// and with WRAP, in a tile that holds the whole level, one past a periodic end
// at the other end.  So no half-sweep has to be followed by a copy of changed
// values to their images, a pass over the ring and a barrier each: 3.4 of 67 us of
// the bottom levels from 16 x 32 on, two fused sweeps of 64 x 128 cells 15.4 against
// 13.5.  (The tile holds zeros on the faces of a high wall.  What is past a wall along the
// axis is read for the face on the wall only, whose equation is not used.)
__device__ __forceinline__ double flip(double x, unsigned m)
{
    return __hiloint2double((int)((unsigned)__double2hiint(x) ^ m), __double2loint(x));
}
__device__ __forceinline__ float flip(float x, unsigned m) { return __uint_as_float(__float_as_uint(x) ^ m); }
template <typename TT, typename R> struct Hood {
    R h[12 * TT::ES];
    __device__ __forceinline__ R *centre() { return h + 4 * TT::ES; }
    template <bool LIN, bool WRAP> __device__ __forceinline__ Ax<TT::ES> load(const R *e, const Ax<TT::ES> &a)
    {
        const bool nl = a.ia == 0, nh = a.ia + 1 == a.ma, tl = a.it == 0, th = a.it + 1 == a.mt;
        // offsets of cells (on) and own faces (fn) along the axis, of cells (ot)
        // and the other axis' faces (ft) across it
        const int wn = WRAP && a.per ? a.ma * a.dn : 0, wt = WRAP && a.pert ? a.mt * a.dt : 0;
        int on[4] = { -a.dn, 0, a.dn, 0 }, fn[4] = { -a.dn, 0, a.dn, 2 * a.dn }, ot[3] = { -a.dt, 0, a.dt }, ft[2] = { 0, a.dt };
        unsigned sl = 0, sh = 0;
        if (nl) on[0] = a.per ? wn - a.dn : 0;
        if (nh) on[2] = a.per ? a.dn - wn : 0;
        if (WRAP) {
            fn[0] = nl && a.per ? wn - a.dn : -a.dn;
            fn[2] = nh ? a.dn - wn : a.dn;
            fn[3] = a.ia + 2 >= a.ma ? 2 * a.dn - wn : 2 * a.dn;
            ft[1] = th ? a.dt - wt : a.dt;
        }
        if (tl) {
            ot[0] = a.pert ? wt - a.dt : 0;
            sl = a.pert ? 0u : 0x80000000u;
        }
        if (th) {
            ot[2] = a.pert ? a.dt - wt : 0;
            sh = a.pert ? 0u : 0x80000000u;
        }
        auto get = [&](int n, int t, int f, int off, int g) {
            h[((n + 1) * 3 + t + 1) * TT::ES + f] = el<TT::ES>(e, off)[g];
        };
#pragma unroll
        for (int n = -1; n <= 1; n++) {
#pragma unroll
            for (int f = T_C; f <= T_MOB; f++) get(n, 0, f, on[n + 1], f);
            if (LIN) {
                get(n, 0, L_DC, on[n + 1], L_DC);
                get(n, 0, L_DRS, on[n + 1], L_DRS);
            }
        }
#pragma unroll
        for (int n = -1; n <= 1; n++)
#pragma unroll
            for (int t = -1; t <= 1; t += 2) {
                get(n, t, T_RN, on[n + 1] + ot[t + 1], T_RN);
                get(n, t, T_MV, on[n + 1] + ot[t + 1], T_MV);
            }
#pragma unroll
        for (int n = -1; n <= 2; n++) {
            get(n, 0, T_U, fn[n + 1], a.fn);
            get(n, 0, T_UN, fn[n + 1], a.fnn);
        }
#pragma unroll
        for (int n = 0; n <= 1; n++) {
            get(n, -1, T_U, fn[n + 1] + ot[0], a.fn);
            get(n, 1, T_U, fn[n + 1] + ot[2], a.fn);
        }
#pragma unroll
        for (int n = -1; n <= 1; n++)
#pragma unroll
            for (int t = 0; t <= 1; t++) {
                get(n, t, T_V, on[n + 1] + ft[t], a.ft);
                get(n, t, T_VN, on[n + 1] + ft[t], a.ftn);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n <= 1; n++) {
            R *lo = h + ((n + 1) * 3) * TT::ES + T_U, *hi = h + ((n + 1) * 3 + 2) * TT::ES + T_U;
            *lo = flip(*lo, sl);
            *hi = flip(*hi, sh);
        }
        Ax<TT::ES> b = a;
        b.dn = 3;
        b.dt = 1;
        b.fn = T_U;
        b.ft = T_V;
        b.fnn = T_UN;
        b.ftn = T_VN;
        return b;
    }
};

// --------------------------------------------------------------------------
// smoother for one cell of the current colour (sec. 7.1), run by a lane pair.
// Segregated (P.coupled = 0): step 1 is Newton on (N_c, N_mu) in (c_ij,
// mubar_ij); step 2 the Vanka box on (uW, uE, vS, vN, p).  Coupled: one Newton
// step on all seven unknowns of the cell with the box equations plus N_c and
// N_mu of the cell.  Its matrix is the 5x5 box matrix bordered by
//   face rows:  dN_f/dc = rho'(c) u_f / (4 dt),  dN_f/dmubar = -a_f / M,
//   mass row:   dN_p/dmubar = alpha Sm / Pe,
//   phase row:  dN_c/du_f = a_f (the advection weights of App. A.5),
//               dN_c/dp = alpha Sm / Pe, Jcc, Jcm,
//   chem. row:  Jmc, Jmm,
// with a_f = rho^n (c^n jump across the face) / (2h), signed along the axis.
// mubar is eliminated first (N_mu; its pivot is Jmm = rho), the rest is solved
// by axes (box_axis, box_solve).
// Velocities come from the tile (the snapshot of this colour); the box faces
// go to unew/vnew, c, mubar, pbar to the level arrays.  In the segregated
// form c, mubar and rho(c) of the cell are also written to the tile between
// the steps (identical values from both lanes), which no other pair of this
// colour reads.
//
// omega relaxes the box's velocity and pressure updates; pomega the
// projection scheme's separate pressure step.
// TO: 0 the results go to the level arrays.  1: the cell sits at tile position
// (ti, tj), which differs from its level position (i, j) at a periodic image,
// and the results stay in the tile; 2: the same in a tile that holds the whole
// level, where the high face of the last cell of a periodic axis is the first
// cell's low face.  In the tile go c, mubar, pbar and rho(c) in place (no other cell of the colour reads
// them), the box faces in the fields T_U2, T_V2 (slot 0; from them to T_U, T_V:
// slot 1), whose elements only this cell's box writes.  AS is the address space of the level arrays and
// right-hand sides (1: global memory, 3: LDS, where the level resides in the
// workgroup's LDS).  HOOD: the neighbourhood is read into registers first.
//
// Against a box assembled and eliminated as a 5x5 matrix, coefficients formed
// per cell and a tile of one array per field, a half-sweep of a finest level
// takes 683 instead of 911 vector instructions per wave and 150 instead of 200
// registers (three waves per SIMD instead of two): 50.4 -> 36 us on 512 x 2048
// (MI355X).

// what a sweep of one cell starts from
template <int ES> struct CellPos {
    Ax<ES> a;
    bool hlo, hhi;    // the lane's faces are unknowns
    size_t k, khi;    // level index of the cell (and its low faces), of the lane's high face
    // where the new high face goes in the tile, from the cell's element
    template <int TO> __device__ __forceinline__ int hi() const
    {
        return TO == 2 && a.ia + 1 == a.ma ? a.dn - a.ma * a.dn : a.dn;
    }
};
template <typename V, typename TT>
__device__ __forceinline__ CellPos<TT::ES> cell_pos(const V &L, const TT &T, int i, int j, int hlf, int slot)
{
    CellPos<TT::ES> c;
    c.a = make_ax(L, T, i, j, hlf, slot);
    c.hlo = c.a.per || c.a.ia >= 1;
    c.hhi = c.a.per || c.a.ia + 1 < c.a.ma;
    c.k = (size_t)j * L.pitch + i;
    const int ihi = hlf ? i : (i + 1 < L.m1 ? i + 1 : 0), jhi = hlf ? (j + 1 < L.m2 ? j + 1 : 0) : j;
    c.khi = (size_t)jhi * L.pitch + ihi;
    return c;
}
// off-diagonal entries of the axis' 2x2 block (a periodic axis of two cells:
// the next face beyond each box face is the box's other face, which so
// enters each face row a second time, through the other cell's advection
// weight and viscosity)
template <typename R, int ES>
__device__ __forceinline__ void box_offdiag(const Kon<R> &K, const R *s, const Ax<ES> &a, bool hlo, bool hhi, R &alh, R &ahl)
{
    const int fnn = a.fnn;
    const R un = s[fnn] + el<ES>(s, a.dn)[fnn];
    const R w = R(4) * (K.ka * (s[T_RN] * un)), vis = R(4) * (K.kv * s[T_MV]);
    alh = hlo ? w - vis : R(0);
    ahl = hhi ? -w - vis : R(0);
    if (a.per && a.ma == 2) {
        const R *o = el<ES>(s, -a.dn);
        const R wo = R(4) * (K.ka * (o[T_RN] * un)), vo = R(4) * (K.kv * o[T_MV]);
        alh = alh - (wo + vo);
        ahl = ahl + (wo - vo);
    }
}

template <int TO, int AS, bool HOOD, typename TT>
__device__ __forceinline__ void relax_pj(const Phys &P, const Kon<double> &K, const View &L, const TT &T, const Rhs &F,
                                         double *unew, double *vnew, int i, int j, int ti, int tj, int hlf,
                                         double omega, double pomega, int slot);

template <bool PJ, int TO, int AS, bool HOOD, typename TT>
__device__ __forceinline__ void relax_cell(const Phys &P, const Kon<double> &K, const View &L, const TT &T,
                                           const Rhs &F, double *unew, double *vnew, int i, int j, int ti, int tj,
                                           int hlf, double omega, double pomega, int slot = 0)
{
    if (PJ) {
        relax_pj<TO, AS, HOOD>(P, K, L, T, F, unew, vnew, i, j, ti, tj, hlf, omega, pomega, slot);
        return;
    }
    constexpr int ES = TT::ES;
    const CellPos<ES> b = cell_pos(L, T, i, j, hlf, slot);
    double *const e = T.at(ti, tj); // results go here, everything is read at s
    Hood<TT, double> H;
    const double *s = e;
    Ax<ES> a = b.a;
    const bool cpl = P.coupled;
    // the right-hand sides first: their loads are then in flight during the
    // cell equations
    const double *fN = face_rhs(F, hlf);
    // (a level in LDS has them; the high face of a wall: loaded, not used)
    double f_c = 0.0, f_mu = 0.0, f_p = 0.0, f_lo = 0.0, f_hi = 0.0;
    if (AS == 3 || F.fc) {
        f_c = lda<AS>(F.fc, b.k);
        f_mu = lda<AS>(F.fmu, b.k);
        f_p = lda<AS>(F.fp, b.k);
        f_lo = lda<AS>(fN, b.k);
        f_hi = lda<AS>(fN, b.khi);
    }
    if (HOOD) {
        a = H.template load<false, TO == 2>(e, b.a);
        s = H.centre();
    }
    double r, drs;
    cell_r(K, s, r, drs);
    const double ulo = s[a.fn], uhi = el<ES>(s, a.dn)[a.fn];
    const CellSum<double> xo = axis_cell<false>(K, s, a, r, drs, ulo, uhi), x = xo + other(xo);
    const CellEq q = cell_eq(K, s, x, r, drs);
    const double r1 = f_c - q.Nc, r2 = f_mu - q.Nmu;
    const double c0 = s[T_C], m0 = s[T_MU], p0 = s[T_P];
    const double Jcp = K.alpha * x.sm; // dN_c/dpbar = dN_p/dmubar
    double bp = f_p - q.Np;
    // coupled box: mubar eliminated by N_mu (pivot Jmm)
    double kmc = 0.0, kbm = 0.0, Jc = 0.0, bc = 0.0, gc = 0.0;
    if (cpl) {
        const double imm = frcp(q.Jmm);
        kmc = q.Jmc * imm;
        kbm = r2 * imm;
        Jc = q.Jcc - q.Jcm * kmc;
        bc = r1 - q.Jcm * kbm;
        gc = 0.5 * K.hidt * drs; // dN_f/dc per unit u_f
    } else {
        // ---- step 1
        const double idet = frcp(q.Jcc * q.Jmm - q.Jcm * q.Jmc);
        const double cnew = c0 + (q.Jmm * r1 - q.Jcm * r2) * idet;
        const double dm = (q.Jcc * r2 - q.Jmc * r1) * idet, mnew = m0 + dm;
        if (!TO && hlf == 0) {
            sta<AS>(L.c, b.k, cnew);
            sta<AS>(L.mu, b.k, mnew);
        }
        const double rnew = rho_of(P, cnew);
        if (HOOD) {
            double *o = H.centre();
            o[T_C] = cnew;
            o[T_MU] = mnew;
            o[T_RS] = rnew;
        }
        if (TO || !HOOD) {
            e[T_C] = cnew;
            e[T_MU] = mnew;
            e[T_RS] = rnew;
        }
        // mass equation with the new mubar of the cell
        bp -= Jcp * dm;
    }
    // ---- the box: this lane's two faces along its axis
    const FaceEq<double> flo = face_eq<double, false, false>(K, s, a), fhi = face_eq<double, false, false>(K, el<ES>(s, a.dn), a);
    const double *P1 = el<ES>(s, a.dn), *M1 = el<ES>(s, -a.dn);
    const double alo = b.hlo ? K.hih * (M1[T_RN] * (s[T_CN] - M1[T_CN])) : 0.0;
    const double ahi = b.hhi ? K.hih * (P1[T_RN] * (P1[T_CN] - s[T_CN])) : 0.0;
    double alh, ahl;
    box_offdiag(K, s, a, b.hlo, b.hhi, alh, ahl);
    const double sb = kbm * K.iM, sc = kmc * K.iM;
    const double blo = b.hlo ? (f_lo - flo.N) + sb * alo : 0.0, bhi = b.hhi ? (f_hi - fhi.N) + sb * ahi : 0.0;
    const double qlo = b.hlo ? gc * ulo + sc * alo : 0.0, qhi = b.hhi ? gc * uhi + sc * ahi : 0.0;
    const BoxAx<double> X = box_axis(b.hlo ? flo.diag : 1.0, b.hhi ? fhi.diag : 1.0, alh, ahl, blo, bhi,
                                     b.hlo ? 1.0 : 0.0, b.hhi ? -1.0 : 0.0, qlo, qhi, alo, ahi);
    double dp, dc, t, tt;
    box_solve(X, box_other(X), cpl, K.kv * s[T_MV], K.kp, K.ih, K.alpha * Jcp, Jcp, kmc, kbm, Jc, bp, bc, dp, dc, t, tt);
    const double nlo = ulo + omega * ((X.xb[0] + t * X.xs[0]) - dc * X.xq[0]);
    const double nhi = uhi + omega * ((X.xb[1] + t * X.xs[1]) - dc * X.xq[1]);
    const double np = p0 + omega * dp;
    if (TO) {
        if (b.hlo) e[b.a.fo] = nlo;
        if (b.hhi) el<ES>(e, b.template hi<TO>())[b.a.fo] = nhi;
        if (hlf == 0) {
            e[T_P] = np;
            if (cpl) {
                e[T_C] = c0 + dc;
                e[T_MU] = m0 + (kbm - kmc * dc);
                e[T_RS] = rho_of(P, c0 + dc);
            }
        }
        return;
    }
    double *fo = hlf ? vnew : unew;
    if (b.hlo) sta<AS>(fo, b.k, nlo);
    if (b.hhi) sta<AS>(fo, b.khi, nhi);
    if (hlf == 0) {
        sta<AS>(L.p, b.k, np);
        if (cpl) {
            sta<AS>(L.c, b.k, c0 + dc);
            sta<AS>(L.mu, b.k, m0 + (kbm - kmc * dc));
        }
    }
}

// the projection scheme's phase and chemical rows, which differ from the
// primitive ones in rho^n (c - c^n)/dt and rho^n mubar ((pj-num-phase),
// (pj-num-chem); the advection at time n+1 is in x.s1)
__device__ __forceinline__ void pj_cell(const Kon<double> &K, const double *s, const CellSum<double> &x, double drs, CellEq &q)
{
    const double rs = s[T_RS], rn = s[T_RN], mu = s[T_MU];
    q.Nc = K.idt * (rn * (s[T_C] - s[T_CN])) + x.s1;
    q.Nmu -= (rs - rn) * mu;
    q.Jcc = K.idt * rn; // and the advection's derivative
    q.Jmm = rn;
    q.Jmc -= drs * mu;
}

// residuals r = f - N(w) of the five equations attached to cell (i,j): the
// cell equations and the momentum equations of its west and south faces (zero
// for a face on a wall), by one lane.  The level and its right-hand sides
// (F.fc NULL: none) are in global memory.
struct Resid {
    double c, mu, p, u, v;
};
// the projection equation (pj-num-pjx) on the face at element s of an axis:
//   u = u~ + dt / A rho (A(rho_ew mubar) D c / M - D pbar / M - grav),
// rho = rho(c) and c, mubar of the iterate, grav = (1/Fr)(A_y rho - rho_ref)
// on north-south faces (gravity acts in the projection equation, as in the
// time-discrete scheme (pj-pj)); zero on a wall face.  ut is u~ on the face;
// w receives 2 dt / (2 A rho).
template <int ES>
__device__ __forceinline__ double face_final(const Kon<double> &K, const double *s, const Ax<ES> &a, bool unk, double ut,
                                             double &w)
{
    const double *L = el<ES>(s, -a.dn);
    const double rL = L[T_RS], rR = s[T_RS], A2 = rL + rR;
    const double st = 0.5 * (rR * L[T_MU] + rL * s[T_MU]) * (s[T_C] - L[T_C]);
    double f = K.kp * (st - (s[T_P] - L[T_P]));
    if (a.hlf) f -= K.inv_Fr * (0.5 * A2 - K.rho_ref);
    w = K.dt2 * frcp(A2);
    return unk ? ut + w * f : 0.0;
}

template <bool PJ, int AS = 1, typename TT>
__device__ __forceinline__ Resid resid_cell(const Kon<double> &K, const View &L, const TT &T, const Rhs &F, int i,
                                            int j)
{
    constexpr int ES = TT::ES;
    const double *e = T.at(i, j);
    const Ax<ES> ax = make_ax(L, T, i, j, 0), ay = make_ax(L, T, i, j, 1);
    const size_t k = (size_t)j * L.pitch + i;
    Resid f = {};
    if (F.fc) f = { lda<AS>(F.fc, k), lda<AS>(F.fmu, k), lda<AS>(F.fp, k), lda<AS>(F.fu, k), lda<AS>(F.fv, k) };
    const bool hu = ax.per || i >= 1, hv = ay.per || j >= 1;
    double ulo = e[T_U], uhi = el<ES>(e, ax.dn)[T_U], vlo = e[T_V], vhi = el<ES>(e, ay.dn)[T_V];
    if (PJ) {
        double w;
        ulo = face_final(K, e, ax, hu, ulo, w);
        uhi = face_final(K, el<ES>(e, ax.dn), ax, ax.per || i + 1 < L.m1, uhi, w);
        vlo = face_final(K, e, ay, hv, vlo, w);
        vhi = face_final(K, el<ES>(e, ay.dn), ay, ay.per || j + 1 < L.m2, vhi, w);
    }
    double r, drs;
    cell_r(K, e, r, drs);
    const CellSum<double> x = axis_cell<PJ>(K, e, ax, r, drs, ulo, uhi) + axis_cell<PJ>(K, e, ay, r, drs, vlo, vhi);
    CellEq q = cell_eq(K, e, x, r, drs);
    if (PJ) pj_cell(K, e, x, drs, q);
    const FaceEq<double> fu = face_eq<double, PJ, false>(K, e, ax), fv = face_eq<double, PJ, false>(K, e, ay);
    return { f.c - q.Nc, f.mu - q.Nmu, f.p - q.Np, hu ? f.u - fu.N : 0.0, hv ? f.v - fv.N : 0.0 };
}

// --------------------------------------------------------------------------
// Projection scheme (sec. 6.2).  The unknowns are c, mubar, pbar and the
// intermediate velocity u~, which the face fields (T_U, T_V) hold during a
// step.  The velocity of time n+1 is eliminated through the projection
// equation (face_final).
//
// Smoother of sec. 7.2 for one cell of the current colour, by a lane pair:
//  1. one Newton step on (N_c, N_mu) in (c, mubar) of the cell, the velocity
//     of time n+1 on its faces held at its value before the update; with the
//     coupled smoother (P.coupled, the default) pbar and the mass equation
//     join this step, the velocity of time n+1 following pbar in its column
//     only;
//  2. the Vanka box of the four intermediate-velocity faces on (pj-num-mx),
//     exact (linear in u~), Jacobi within the colour;
//  3. one Newton step in pbar on the mass equation (pj-num-mass) with the
//     velocity of time n+1 from the new u~, c, mubar (exact: linear in pbar);
//  4. the velocity of time n+1 is never stored, so nothing is left to update.
// The tile entries of the cell (c, mubar, rho(c)) are updated after step 1; no
// other pair of this colour reads them.
template <int TO, int AS, bool HOOD, typename TT>
__device__ __forceinline__ void relax_pj(const Phys &P, const Kon<double> &K, const View &L, const TT &T, const Rhs &F,
                                         double *unew, double *vnew, int i, int j, int ti, int tj, int hlf,
                                         double omega, double pomega, int slot)
{
    constexpr int ES = TT::ES;
    const CellPos<ES> b = cell_pos(L, T, i, j, hlf, slot);
    double *const e = T.at(ti, tj); // results go here, everything is read at s
    Hood<TT, double> H;
    double *s = e;
    Ax<ES> a = b.a;
    const double *fN = face_rhs(F, hlf);
    // (a level in LDS has them; the high face of a wall: loaded, not used)
    double f_c = 0.0, f_mu = 0.0, f_p = 0.0, f_lo = 0.0, f_hi = 0.0;
    if (AS == 3 || F.fc) {
        f_c = lda<AS>(F.fc, b.k);
        f_mu = lda<AS>(F.fmu, b.k);
        f_p = lda<AS>(F.fp, b.k);
        f_lo = lda<AS>(fN, b.k);
        f_hi = lda<AS>(fN, b.khi);
    }
    if (HOOD) {
        a = H.template load<false, TO == 2>(e, b.a);
        s = H.centre();
    }
    const double *P1 = el<ES>(s, a.dn), *M1 = el<ES>(s, -a.dn);
    // ---- step 1
    double wlo, whi;
    const double ulo0 = face_final(K, s, a, b.hlo, s[a.fn], wlo);
    const double uhi0 = face_final(K, P1, a, b.hhi, P1[a.fn], whi);
    double r, drs;
    cell_r(K, s, r, drs);
    const CellSum<double> xo = axis_cell<true>(K, s, a, r, drs, ulo0, uhi0), x = xo + other(xo);
    CellEq q = cell_eq(K, s, x, r, drs);
    pj_cell(K, s, x, drs, q);
    const double dax = K.hih * (M1[T_RS] * ulo0 - P1[T_RS] * uhi0);
    q.Jcc += dax + other(dax);
    const double c0 = s[T_C], m0 = s[T_MU], p0 = s[T_P];
    const double r1 = f_c - q.Nc, r2 = f_mu - q.Nmu;
    const double Jpm = K.alpha * x.sm;
    double dc, dm, pnew = p0;
    if (P.coupled) {
        // pbar joins the step with the mass equation: its column lets the
        // velocity of time n+1 follow pbar through (pj-num-pjx) (on the lo
        // face D pbar falls by pbar/h, on the hi face it rises), the c and
        // mubar columns hold it
        const double dlo = b.hlo ? -K.kp * wlo : 0.0, dhi = b.hhi ? K.kp * whi : 0.0;
        const double cl = K.hih * (M1[T_RS] * (c0 - M1[T_C]) * dlo + P1[T_RS] * (P1[T_C] - c0) * dhi);
        const double jx = K.ih * (dhi - dlo);
        const double Jcp = cl + other(cl) + Jpm, Jpp = jx + other(jx) + K.alpha * Jpm;
        const double r3 = f_p - q.Np;
        // eliminate pbar by the mass row (pivot Jpp), then mubar by the
        // chemical row (pivot Jmm): a 2x2 system in c and mubar remains
        const double ipp = frcp(Jpp);
        const double kcm = q.Jcm - Jcp * Jpm * ipp, rc1 = r1 - Jcp * r3 * ipp;
        const double idet = frcp(q.Jcc * q.Jmm - kcm * q.Jmc);
        dc = (q.Jmm * rc1 - kcm * r2) * idet;
        dm = (q.Jcc * r2 - q.Jmc * rc1) * idet;
        pnew = p0 + (r3 - Jpm * dm) * ipp;
        s[T_P] = pnew;
    } else {
        const double idet = frcp(q.Jcc * q.Jmm - q.Jcm * q.Jmc);
        dc = (q.Jmm * r1 - q.Jcm * r2) * idet;
        dm = (q.Jcc * r2 - q.Jmc * r1) * idet;
    }
    const double cnew = c0 + dc, mnew = m0 + dm;
    if (!TO && hlf == 0) {
        sta<AS>(L.c, b.k, cnew);
        sta<AS>(L.mu, b.k, mnew);
    }
    // (with the neighbourhood in registers, s is not the tile's element)
    s[T_C] = cnew;
    s[T_MU] = mnew;
    s[T_RS] = rho_of(P, cnew);
    if (HOOD && TO) {
        e[T_C] = cnew;
        e[T_MU] = mnew;
        e[T_RS] = s[T_RS];
    }
    // ---- step 2: the intermediate-velocity box; the axes couple through the
    // viscous terms alone: V x = b + s gd D_o
    const FaceEq<double> flo = face_eq<double, true, false>(K, s, a), fhi = face_eq<double, true, false>(K, P1, a);
    double alh, ahl;
    box_offdiag(K, s, a, b.hlo, b.hhi, alh, ahl);
    const double gd = K.kv * s[T_MV];
    const BoxAx<double> X = box_axis(b.hlo ? flo.diag : 1.0, b.hhi ? fhi.diag : 1.0, alh, ahl,
                                     b.hlo ? f_lo - flo.N : 0.0, b.hhi ? f_hi - fhi.N : 0.0, b.hlo ? 1.0 : 0.0,
                                     b.hhi ? -1.0 : 0.0, 0.0, 0.0, 0.0, 0.0);
    const double oDb = other(X.Db), oDs = other(X.Ds);
    const double gx = gd * X.Ds, gy = gd * oDs;
    const double t = gd * ((oDb + gy * X.Db) * frcp(1.0 - gx * gy));
    const double ut0 = s[a.fn], ut1 = P1[a.fn];
    const double ulo = ut0 + omega * (X.xb[0] + t * X.xs[0]), uhi = ut1 + omega * (X.xb[1] + t * X.xs[1]);
    if (TO) {
        if (b.hlo) e[b.a.fo] = ulo;
        if (b.hhi) el<ES>(e, b.template hi<TO>())[b.a.fo] = uhi;
    } else {
        double *fo = hlf ? vnew : unew;
        if (b.hlo) sta<AS>(fo, b.k, ulo);
        if (b.hhi) sta<AS>(fo, b.khi, uhi);
    }
    // ---- step 3: pbar from the mass equation with the new u~ (passed by
    // value: the tile keeps the snapshot that other boxes of this colour read)
    const double ulo1 = face_final(K, s, a, b.hlo, ulo, wlo), uhi1 = face_final(K, P1, a, b.hhi, uhi, whi);
    const double jax = (K.ih * K.kp) * ((b.hlo ? wlo : 0.0) + (b.hhi ? whi : 0.0));
    const double dv = K.ih * ((uhi1 - ulo1) - (uhi0 - ulo0));
    const double Np = q.Np + (dv + other(dv)) + Jpm * (dm + K.alpha * (pnew - p0));
    const double Jp = jax + other(jax) + K.alpha * Jpm;
    if (hlf == 0) {
        const double pf = pnew + pomega * (f_p - Np) * frcp(Jp);
        if (TO) e[T_P] = pf;
        else sta<AS>(L.p, b.k, pf);
    }
}

} // namespace qn
