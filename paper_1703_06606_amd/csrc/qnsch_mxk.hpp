// qnsch_mxk.hpp -- work-list kernels of the mixed-precision step: one FP32
// multigrid V-cycle on the correction equation J(w^) delta = r (see
// qnsch_lin.hpp), with the FP64 residual, update and reductions done by the
// kernels of qnsch_kern.hpp.
//
// Correction cycle on a hierarchy of levels (the coarse-grid correction
// scheme for a linear problem; sec. 7.1 gives the smoother and transfers):
//   smooth (nu1 red-black sweeps), restrict r - J delta and the linearisation
//   point to the next level with delta_H = 0, recurse, solve the coarsest
//   level in LDS, prolongate delta_H and add it, smooth (nu2 sweeps);
// then w += delta in FP64.  The coarse operators are the rediscretised
// Jacobians J_H(R w^).
#pragma once
#include "qnsch_kern.hpp"

namespace qn {

#define LTILE_FLOATS (L_ES * TILE_S * (TY + 3))
static_assert(LTILE_FLOATS * 4 <= 65536, "FP32 tile exceeds 64 KiB of LDS");

__device__ __forceinline__ LView lview_of(const Desc &d, int par)
{
    LView V;
    V.c = d.xc; V.mu = d.xmu; V.u = d.xu; V.v = d.xv;
    V.dc = d.dc; V.dmu = d.dmu; V.dp = d.dp;
    V.du = d.dub[par]; V.dv = d.dvb[par];
    V.cn = d.cnf; V.un = d.unf; V.vn = d.vnf;
    V.rc = d.rc; V.rmu = d.rmu; V.rp = d.rp; V.ru = d.ru; V.rv = d.rv;
    V.m1 = d.m1; V.m2 = d.m2; V.pitch = d.pitch;
    V.bcx = d.bcx; V.bcy = d.bcy;
    return V;
}

// one colour half-sweep of the correction smoother; the correction faces are
// read from buffer par and written to par^1
template <typename IT> __device__ __forceinline__ void k_mx_halfsweep_body(const IT &it, int colour, float omega)
{
    TILE_LDS float sm[LTILE_FLOATS];
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    if (!tile_valid(it, k, d)) return;
    const int par = it_par(it, k);
    const LView L = lview_of(d, par);
    const TileF T = item_tile<TileF>(sm, it, k, d);
    ltile_load<2, TBLK>(d.Pf, L, T);
    __syncthreads();
    const int pr = threadIdx.x >> 1, hlf = threadIdx.x & 1;
    const int lj = pr / (TX / 2), kk = pr - lj * (TX / 2);
    const int j = T.j0 + lj;
    const int i = T.i0 + 2 * kk + ((j + colour) & 1);
    if (i < L.m1 && j < L.m2) lrelax_cell<0, 1, false>(d.Pf, d.Kf, L, T, d.dub[par ^ 1], d.dvb[par ^ 1], i, j, i, j, hlf, omega);
}
QN_KERNEL(k_mx_halfsweep, HS_ATTR, (int colour, float omega), (colour, omega))
// finest-level launches under their own name (profiles)
template <typename IT> __device__ __forceinline__ void k_mx_halfsweep_fine_body(const IT &it, int colour, float omega)
{
    k_mx_halfsweep_body(it, colour, omega);
}
QN_KERNEL(k_mx_halfsweep_fine, HS_ATTR, (int colour, float omega), (colour, omega))

// P delta_H of the FP32 correction: cells piecewise constant, faces as in
// prolong_load / prolong_apply (a face on a wall is no unknown), in two parts
// so that every load is in flight before any value is used.  The coarse
// arrays are read from the descriptor once per workgroup, through a global
// pointer (scalar loads).
struct PSrcF {
    const float *dc, *dmu, *dp, *du, *dv;
    int pitch, m1, m2, bcx, bcy;
};
__device__ __forceinline__ PSrcF psrcf_of(const Desc &d, const Desc *cp, int cpar)
{
    const __attribute__((address_space(1))) Desc &C = *(const __attribute__((address_space(1))) Desc *)cp;
    PSrcF s;
    s.dc = C.dc; s.dmu = C.dmu; s.dp = C.dp; s.du = C.dub[cpar]; s.dv = C.dvb[cpar];
    s.pitch = C.pitch; s.m1 = C.m1; s.m2 = C.m2; s.bcx = d.bcx; s.bcy = d.bcy;
    return s;
}
// the coarse cell of fine cell (ic, jc), and for the fine faces (iu, ju), (iv,
// jv) the coarse face each lies on and the next one east (north): the periodic
// image, or, where there is none, the same face again (loaded, not used)
struct PRawF {
    float c, mu, p, u[2], v[2];
};
__device__ __forceinline__ PRawF mx_prolong_load(const PSrcF &C, int ic, int jc, int iu, int ju, int iv, int jv)
{
    PRawF r;
    const size_t kc = (size_t)(jc >> 1) * C.pitch + (ic >> 1);
    r.c = lda<1>(C.dc, kc); r.mu = lda<1>(C.dmu, kc); r.p = lda<1>(C.dp, kc);
    {
        const int I = iu >> 1, J = ju >> 1;
        const size_t k0 = (size_t)J * C.pitch + I, k1 = I + 1 < C.m1 ? k0 + 1 : (C.bcx ? (size_t)J * C.pitch : k0);
        r.u[0] = lda<1>(C.du, k0); r.u[1] = lda<1>(C.du, k1);
    }
    {
        const int I = iv >> 1, J = jv >> 1;
        const size_t k0 = (size_t)J * C.pitch + I, k1 = J + 1 < C.m2 ? k0 + C.pitch : (C.bcy ? (size_t)I : k0);
        r.v[0] = lda<1>(C.dv, k0); r.v[1] = lda<1>(C.dv, k1);
    }
    return r;
}
// ... the corrections of the u face in column iu and the v face in row jv
// (zero for a face on a wall)
__device__ __forceinline__ void mx_prolong_apply(const PSrcF &C, const PRawF &r, int iu, int jv, float &du, float &dv)
{
    du = r.u[0];
    if (iu & 1) {
        const float e = ((iu >> 1) + 1 < C.m1 || C.bcx) ? r.u[1] : 0.0f;
        du = 0.5f * (du + e);
    }
    if (!(C.bcx || iu >= 1)) du = 0.0f;
    dv = r.v[0];
    if (jv & 1) {
        const float e = ((jv >> 1) + 1 < C.m2 || C.bcy) ? r.v[1] : 0.0f;
        dv = 0.5f * (dv + e);
    }
    if (!(C.bcy || jv >= 1)) dv = 0.0f;
}

// temporal blocking of the correction smoother: NS sweeps per launch, as
// fused_body (the widened tile in LDS, the cell corrections from one set to the
// other, the face corrections from buffer par to par ^ 1; the first sweep
// of a post-smoothing takes P delta_H as it loads the level)
template <bool prolong>
__device__ __forceinline__ void mx_fused_load(const PhysF &P, const LView &L, const TileF &T, const PSrcF &pc)
{
    const int n = T.W * T.H;
    for (int e = threadIdx.x; e < n; e += FUSED_BLK(false)) {
        const int b = e / T.W, a = e - b * T.W;
        int i = T.i0 - 1 + a, j = T.j0 - 1 + b;
        if (L.bcx) i = wrapi(i, L.m1);
        if (L.bcy) j = wrapi(j, L.m2);
        const TileSrc q = tile_src(L.m1, L.m2, L.pitch, L.bcx, L.bcy, i, j);
        if (q.sc == 0) {
            tile_zero(T, b * T.S + a);
            continue;
        }
        // the level is in global memory; every load before any use
        float v[9] = { lda<1>(L.c, q.c), lda<1>(L.dc, q.c), lda<1>(L.dmu, q.c), lda<1>(L.dp, q.c), lda<1>(L.du, q.u),
                       lda<1>(L.dv, q.v), lda<1>(L.cn, q.c), lda<1>(L.un, q.u), lda<1>(L.vn, q.v) };
        PRawF raw = {};
        int iu = 0, jv = 0;
        if (prolong) {
            iu = q.u % L.pitch;
            jv = q.v / L.pitch;
            raw = mx_prolong_load(pc, q.c % L.pitch, q.c / L.pitch, iu, q.u / L.pitch, q.v % L.pitch, jv);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (prolong) {
            float du, dv;
            mx_prolong_apply(pc, raw, iu, jv, du, dv);
            v[1] += raw.c;
            v[2] += raw.mu;
            v[3] += raw.p;
            if (q.su) v[4] += du;
            if (q.sv) v[5] += dv;
        }
        float *s = T.s + (b * T.S + a) * L_ES;
        ltile_put(P, s, q.su, q.sv, v);
        s[T_U2] = s[T_U];
        s[T_V2] = s[T_V];
    }
}
template <int NS, int TS> __device__ __forceinline__ void mx_fused_body(const Item1 &it, int dir, float omega, int prolong)
{
    typedef Fused<NS, TS> G;
    extern __shared__ __attribute__((aligned(16))) float smf[];
    const Desc &d = *it.d;
    int i0, j0; // of the tile
    if (!item_tile_at<TS>(it, 0, d, i0, j0)) return;
    const PhysF P = d.Pf;
    const Kon<float> K = d.Kf;
    const int par = it_par(it, 0);
    LView L = lview_of(d, par);
    LView O = L;
    if (dir) {
        L.dc = d.dc2; L.dmu = d.dmu2; L.dp = d.dp2;
    } else {
        O.dc = d.dc2; O.dmu = d.dmu2; O.dp = d.dp2;
    }
    TileF T;
    T.s = smf; T.i0 = i0 - G::EXT; T.j0 = j0 - G::EXT; T.W = G::W; T.H = G::W; T.S = G::S;
    float *const un = d.dub[par ^ 1], *const vn = d.dvb[par ^ 1];
    if (prolong) mx_fused_load<true>(P, L, T, psrcf_of(d, &d + 1, it_cpar(it, 0)));
    else mx_fused_load<false>(P, L, T, PSrcF());
    __syncthreads();
    const int hlf = threadIdx.x & 1;
    auto half = [&](auto cext, auto ccol) {
        constexpr int ext = cext.value, colour = ccol.value, w = TS + 2 * ext;
        for (int pr = threadIdx.x >> 1; pr < w * w / 2; pr += FUSED_BLK(false) / 2) {
            const int lj = pr / (w / 2), kk = pr - lj * (w / 2);
            const int tj = j0 - ext + lj, ti = i0 - ext + 2 * kk + ((tj + colour) & 1);
            if ((L.bcx || (ti >= 0 && ti < L.m1)) && (L.bcy || (tj >= 0 && tj < L.m2))) {
                const int i = L.bcx ? wrapi(ti, L.m1) : ti, j = L.bcy ? wrapi(tj, L.m2) : tj;
                lrelax_cell<1, 1, true>(P, K, L, T, nullptr, nullptr, i, j, ti, tj, hlf, omega, colour);
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
        const int pr = threadIdx.x >> 1, lj = pr / (TS / 2), kk = pr - lj * (TS / 2);
        const int j = j0 + lj, i = i0 + 2 * kk + ((j + 1) & 1);
        if (i < L.m1 && j < L.m2) lrelax_cell<0, 1, true>(P, K, O, T, un, vn, i, j, i, j, hlf, omega, 1);
    } else if (threadIdx.x < 2 * TS * TS) {
        const int q = (threadIdx.x - TS * TS) >> 1, lj = q / (TS / 2), kk = q - lj * (TS / 2);
        const int j = j0 + lj, i = i0 + 2 * kk + (j & 1);
        if (i < L.m1 && j < L.m2) {
            const float *e = T.at(i, j);
            const size_t g = (size_t)j * L.pitch + i;
            if (hlf == 0) {
                sta<1>(O.dc, g, e[L_DC]);
                sta<1>(O.dmu, g, e[T_MU]);
            } else {
                sta<1>(O.dp, g, e[T_P]);
            }
        }
    }
}
__device__ __forceinline__ void k_mx_fused_body(const Item1 &it, int dir, float omega, int prolong)
{
    mx_fused_body<1, 16>(it, dir, omega, prolong);
}
QN_KERNEL1(k_mx_fused, __launch_bounds__(FUSED_BLK(false)), (int dir, float omega, int prolong), (dir, omega, prolong))
__device__ __forceinline__ void k_mx_fused2_body(const Item1 &it, int dir, float omega, int prolong)
{
    mx_fused_body<2, 8>(it, dir, omega, prolong);
}
QN_KERNEL1(k_mx_fused2, __launch_bounds__(FUSED_BLK(false)), (int dir, float omega, int prolong), (dir, omega, prolong))

// r - J delta on the item's level, restricted to the next coarser level
// (cells: mean of four; faces: mean of the two coincident fine faces),
// together with the linearisation point; the coarse correction starts at 0
// (one lane per fine cell, a coarse cell's children in a quad of lanes)
__device__ __forceinline__ float quad_sum(float x)
{
    x += other(x);
    return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, false));
}
template <typename IT> __device__ __forceinline__ void k_mx_restrict_body(const IT &it, int set)
{
    TILE_LDS float sm[L_ES * TILE_S * (TY + 2)];
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    if (!tile_valid(it, k, d)) return;
    const Desc &C = (&d)[1];
    LView Lf = lview_of(d, it_par(it, k));
    if (set) { // the pre-smoothing left the cell corrections in the second set
        Lf.dc = d.dc2; Lf.dmu = d.dmu2; Lf.dp = d.dp2;
    }
    const TileF T = item_tile<TileF, TX + 2>(sm, it, k, d);
    ltile_load<2, TBLK>(d.Pf, Lf, T);
    __syncthreads();
    const int cc = threadIdx.x >> 2, ch = threadIdx.x & 3;
    const int I = T.i0 / 2 + cc % (TX / 2), J = T.j0 / 2 + cc / (TX / 2);
    const int i = 2 * I + (ch & 1), j = 2 * J + (ch >> 1);
    if (I >= C.m1 || J >= C.m2) return; // a quad's lanes share I, J
    const size_t w = (size_t)j * Lf.pitch + i;
    const float xmu = lda<1>(Lf.mu, w), xu = lda<1>(Lf.u, w), xv = lda<1>(Lf.v, w);
    const ResidF r = lresid_cell(d.Kf, Lf, T, i, j);
    const bool wu = (ch & 1) == 0, wv = (ch >> 1) == 0; // faces of the coarse cell
    const float rc = quad_sum(r.c), rm = quad_sum(r.mu), rp = quad_sum(r.p), ru = quad_sum(wu ? r.u : 0.0f),
                rv = quad_sum(wv ? r.v : 0.0f);
    const float sc = quad_sum(T.q(T_C, i, j)), smu = quad_sum(xmu), su = quad_sum(wu ? xu : 0.0f),
                sv = quad_sum(wv ? xv : 0.0f);
    const size_t q = (size_t)J * C.pitch + I;
    const int cp = it_cpar(it, k);
    if (ch == 0) {
        sta<1>(C.xc, q, 0.25f * sc);
        sta<1>(C.xmu, q, 0.25f * smu);
        sta<1>(C.xu, q, 0.5f * su);
        sta<1>(C.xv, q, 0.5f * sv);
    } else if (ch == 1) {
        sta<1>(C.rc, q, 0.25f * rc);
        sta<1>(C.rmu, q, 0.25f * rm);
        sta<1>(C.rp, q, 0.25f * rp);
        sta<1>(C.ru, q, 0.5f * ru);
        sta<1>(C.rv, q, 0.5f * rv);
    } else if (ch == 2) {
        sta<1>(C.dc, q, 0.0f);
        sta<1>(C.dmu, q, 0.0f);
        sta<1>(C.dp, q, 0.0f);
    } else {
        sta<1>(C.dub[cp], q, 0.0f);
        sta<1>(C.dvb[cp], q, 0.0f);
    }
}
QN_KERNEL(k_mx_restrict, __launch_bounds__(TBLK), (int set), (set))

// delta_h += P delta_H, one thread per fine cell
template <typename IT> __device__ __forceinline__ void k_mx_prolong_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= d.m1 * d.m2) return;
    const int j = t / d.m1, i = t - j * d.m1;
    const size_t kf = (size_t)j * d.pitch + i;
    const PSrcF ps = psrcf_of(d, &d + 1, it_cpar(it, k));
    float *ub = d.dub[it_par(it, k)], *vb = d.dvb[it_par(it, k)];
    const PRawF raw = mx_prolong_load(ps, i, j, i, j, i, j);
    const float c0 = lda<1>(d.dc, kf), m0 = lda<1>(d.dmu, kf), p0 = lda<1>(d.dp, kf), u0 = lda<1>(ub, kf),
                v0 = lda<1>(vb, kf);
    __builtin_amdgcn_sched_barrier(0);
    float du, dv;
    mx_prolong_apply(ps, raw, i, j, du, dv);
    sta<1>(d.dc, kf, c0 + raw.c);
    sta<1>(d.dmu, kf, m0 + raw.mu);
    sta<1>(d.dp, kf, p0 + raw.p);
    if (ps.bcx || i >= 1) sta<1>(ub, kf, u0 + du);
    if (ps.bcy || j >= 1) sta<1>(vb, kf, v0 + dv);
}
QN_KERNEL(k_mx_prolong, __launch_bounds__(BLK), (), ())

// The bottom of the correction cycle, as k_bottom: a level and every coarser
// one resident in LDS in one workgroup per item (the correction and the
// linearisation point of the coarser levels never leave it).  LDS of a level:
// its tile, the right-hand sides and the linearisation point's mubar, u, v,
// the images.
struct BotLevF {
    float *r, *x; // 5 and 3 fields of m1*m2
    Image *ring;
    TileF T;
    int m1, m2;
};
__host__ __device__ inline size_t bot_floats(int m1, int m2)
{
    return bot_tile(m1, m2, L_ES) + (size_t)8 * m1 * m2 + 4 * (size_t)ring_size(m1, m2);
}
__device__ __forceinline__ BotLevF bot_lev(float *sm, int m1, int m2, int l)
{
    int off = 0; // in 16 bytes
    for (; l > 0; l--) {
        off += (int)(bot_floats(m1, m2) / 4);
        m1 >>= 1;
        m2 >>= 1;
    }
    sm += 4 * off;
    BotLevF B;
    B.m1 = m1; B.m2 = m2;
    B.T.s = sm; B.T.i0 = 0; B.T.j0 = 0; B.T.W = m1 + 3; B.T.H = m2 + 3; B.T.S = bot_stride(m1);
    B.r = sm + bot_tile(m1, m2, L_ES);
    B.x = B.r + 5 * m1 * m2;
    B.ring = (Image *)(B.x + 3 * m1 * m2);
    return B;
}
__device__ __forceinline__ LView bot_view(const BotLevF &B, const Desc &d)
{
    const int n = B.m1 * B.m2;
    LView L = {};
    L.m1 = B.m1; L.m2 = B.m2; L.pitch = B.m1;
    L.bcx = d.bcx; L.bcy = d.bcy;
    L.mu = B.x; L.u = B.x + n; L.v = B.x + 2 * n;
    L.rc = B.r; L.rmu = B.r + n; L.rp = B.r + 2 * n; L.ru = B.r + 3 * n; L.rv = B.r + 4 * n;
    return L;
}
__device__ __forceinline__ void bot_images(const BotLevF &B, int t)
{
    const int n = ring_size(B.m1, B.m2);
    for (int k = t; k < n; k += BOT) {
        const Image g = B.ring[k];
        const float *s = B.T.s + g.c * L_ES;
        const float dc = s[L_DC], mu = s[T_MU], p = s[T_P], drs = s[L_DRS];
        const float u = B.T.s[(g.u >> 2) * L_ES + T_U], v = B.T.s[(g.v >> 2) * L_ES + T_V];
        float *t = B.T.s + g.e * L_ES;
        t[L_DC] = dc;
        t[T_MU] = mu;
        t[T_P] = p;
        t[L_DRS] = drs;
        t[T_U] = signed_val((g.u & 3) - 1, u);
        t[T_V] = signed_val((g.v & 3) - 1, v);
    }
}
__device__ __forceinline__ void bot_smooth(const PhysF &P, const Desc &d, const BotLevF &B, int sweeps, float omega)
{
    const Kon<float> K = d.Kf;
    const LView L = bot_view(B, d);
    const int half = B.m1 >> 1, n2 = 2 * half * B.m2, pr = threadIdx.x >> 1, hlf = threadIdx.x & 1;
    const int j0 = pr / half, i0 = 2 * (pr - j0 * half), dj = (BOT / 2) / half, di = 2 * ((BOT / 2) - dj * half);
    auto sweep = [&](auto colour) {
        int i = i0, j = j0;
        for (int t = threadIdx.x; t < n2; t += BOT) {
            const int ic = i + ((j + colour.value) & 1);
            lrelax_cell<2, 3, true>(P, K, L, B.T, nullptr, nullptr, ic, j, ic, j, hlf, omega, colour.value);
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
// residual of level A and the linearisation point restricted to the next level
// C, whose correction starts at zero (its time-n fields are in the tile)
__device__ __forceinline__ void bot_restrict(const PhysF &P, const Desc &d, const BotLevF &A, const BotLevF &C)
{
    const int nc = C.m1 * C.m2, na = A.m1 * A.m2, rt = BOT - 1 - threadIdx.x;
    for (int t = rt; t < nc; t += BOT) {
        const int J = t / C.m1, I = t - J * C.m1, w = 2 * J * A.m1 + 2 * I;
        const float *a = A.T.at(2 * I, 2 * J), *b = a + L_ES, *s = el<L_ES>(a, A.T.S), *e = s + L_ES;
        const float *x = A.x + w, *y = x + A.m1;
        const float c = 0.25f * ((a[T_C] + b[T_C]) + (s[T_C] + e[T_C]));
        const float xm = 0.25f * ((x[0] + x[1]) + (y[0] + y[1])), xu = 0.5f * (x[na] + y[na]), xv = 0.5f * (x[2 * na] + x[2 * na + 1]);
        float *o = C.T.at(I, J);
        o[T_C] = c;
        o[T_RS] = rhof(P, c);
        o[T_MU] = o[T_P] = o[L_DC] = o[L_DRS] = 0.0f;
        o[T_U] = o[T_U2] = o[T_V] = o[T_V2] = 0.0f;
        C.x[t] = xm;
        C.x[nc + t] = xu;
        C.x[2 * nc + t] = xv;
    }
    bot_images(A, threadIdx.x);
    __syncthreads();
    // images: also of the linearisation point's c and rho, once
    const int n = ring_size(C.m1, C.m2);
    for (int k = rt; k < n; k += BOT) {
        const Image g = C.ring[k];
        const float *s = C.T.s + g.c * L_ES;
        float *t = C.T.s + g.e * L_ES;
        t[T_C] = s[T_C];
        t[T_RS] = s[T_RS];
    }
    const Kon<float> K = d.Kf;
    const LView L = bot_view(A, d);
    for (int t = threadIdx.x; t < 4 * nc; t += BOT) {
        const int cc = t >> 2, ch = t & 3;
        const int J = cc / C.m1, I = cc - J * C.m1, i = 2 * I + (ch & 1), j = 2 * J + (ch >> 1);
        const ResidF r = lresid_cell<3>(K, L, A.T, i, j);
        const bool wu = (ch & 1) == 0, wv = (ch >> 1) == 0; // faces of the coarse cell
        const float f[5] = { 0.25f * quad_sum(r.c), 0.25f * quad_sum(r.mu), 0.25f * quad_sum(r.p),
                             0.5f * quad_sum(wu ? r.u : 0.0f), 0.5f * quad_sum(wv ? r.v : 0.0f) };
        if (ch == 0)
#pragma unroll
            for (int q = 0; q < 5; q++) C.r[q * nc + cc] = f[q];
    }
    __syncthreads();
}
// delta_A += P delta_C (k_mx_prolong's arithmetic)
__device__ __forceinline__ void bot_prolong(const PhysF &P, const Desc &d, const BotLevF &A, const BotLevF &C)
{
    const int na = A.m1 * A.m2;
    const bool bx = d.bcx, by = d.bcy;
    for (int t = threadIdx.x; t < na; t += BOT) {
        const int j = t / A.m1, i = t - j * A.m1, I = i >> 1, J = j >> 1;
        const float *s = C.T.at(I, J);
        const bool ix = I + 1 < C.m1, jy = J + 1 < C.m2;
        const float u0 = s[T_U], u1 = C.T.at(ix ? I + 1 : 0, J)[T_U], v0 = s[T_V], v1 = C.T.at(I, jy ? J + 1 : 0)[T_V];
        const float du = i & 1 ? 0.5f * (u0 + (ix || bx ? u1 : 0.0f)) : u0, dv = j & 1 ? 0.5f * (v0 + (jy || by ? v1 : 0.0f)) : v0;
        float *o = A.T.at(i, j);
        const float dc = o[L_DC] + s[L_DC], rs = o[T_RS];
        o[L_DC] = dc;
        o[L_DRS] = -P.alpha * rs * rs * dc;
        o[T_MU] += s[T_MU];
        o[T_P] += s[T_P];
        if (bx || i >= 1) o[T_U] += du;
        if (by || j >= 1) o[T_V] += dv;
    }
    __syncthreads();
}
template <typename IT>
__device__ __forceinline__ void k_mx_bottom_body(const IT &it, int nu1, int nu2, int nuc, float omega, float comega)
{
    extern __shared__ __attribute__((aligned(16))) float smf[];
    const int k = find_item(it);
    if ((int)blockIdx.x != it_start(it, k)) return; // pads the list (k_bottom)
    const Desc &d = it_desc(it, k);
    const PhysF P = d.Pf;
    const int par = it_par(it, k), m1 = d.m1, m2 = d.m2, depth = d.depth;
    const LView L = lview_of(d, par);
    float *const ua = d.dub[par], *const va = d.dvb[par];
    const int n = m1 * m2;
    int lc = 1, ec = threadIdx.x;
    const bool hc = bot_find(lc, ec, depth, m1, m2, [](int a, int b) { return a * b; });
    auto lev = [&](int l) { return bot_lev(smf, m1, m2, l); };
    const BotLevF Bc = lev(hc ? lc : 0);
    const int jc = ec / Bc.m1, ic = ec - jc * Bc.m1;
    const Desc &dc = (&d)[hc ? lc : 0];
    const float *const pc = dc.cnf, *const pu = dc.unf, *const pv = dc.vnf;
    {
        const BotLevF B = bot_lev(smf, m1, m2, 0);
        for (int t0 = threadIdx.x; t0 < n || t0 < BOT; t0 += BOT) {
            const int e = min(t0, n - 1), j = e / m1, i = e - j * m1;
            const TileSrc q = tile_src(m1, m2, L.pitch, L.bcx, L.bcy, i, j);
            const float v[9] = { lda<1>(L.c, q.c), lda<1>(L.dc, q.c), lda<1>(L.dmu, q.c), lda<1>(L.dp, q.c),
                                 lda<1>(L.du, q.u), lda<1>(L.dv, q.v), lda<1>(L.cn, q.c), lda<1>(L.un, q.u),
                                 lda<1>(L.vn, q.v) };
            const float f[8] = { lda<1>(L.rc, q.c), lda<1>(L.rmu, q.c), lda<1>(L.rp, q.c), lda<1>(L.ru, q.c),
                                 lda<1>(L.rv, q.c), lda<1>(L.mu, q.c), lda<1>(L.u, q.c), lda<1>(L.v, q.c) };
            const bool co = hc && t0 < BOT;
            float w[3] = { 0.0f, 0.0f, 0.0f };
            TileSrc qc = {};
            if (co) {
                qc = tile_src(Bc.m1, Bc.m2, Bc.m1, L.bcx, L.bcy, ic, jc);
                w[0] = lda<1>(pc, qc.c); w[1] = lda<1>(pu, qc.u); w[2] = lda<1>(pv, qc.v);
            }
            if (t0 < BOT)
                bot_rings(depth, m1, m2, lev, [&](const BotLevF &R, int k) { R.ring[k] = ring_entry(R.T, R.m1, R.m2, L.bcx, L.bcy, k); });
            __builtin_amdgcn_sched_barrier(0);
            if (t0 < n) {
                float *t = B.T.at(i, j);
                ltile_put(P, t, q.su, q.sv, v);
                t[T_U2] = t[T_U];
                t[T_V2] = t[T_V];
#pragma unroll
                for (int g = 0; g < 8; g++) B.r[g * n + e] = f[g]; // r, then x
            }
            if (co) {
                float *o = Bc.T.at(ic, jc);
                o[T_CN] = w[0];
                o[T_RN] = rhof(P, w[0]);
                o[T_MV] = viscf(P, w[0]);
                o[T_MOB] = mobf(P, w[0]);
                o[T_UN] = signed_val(qc.su, w[1]);
                o[T_VN] = signed_val(qc.sv, w[2]);
            }
        }
    }
    __syncthreads();
    bot_rings(depth, m1, m2, lev, [&](const BotLevF &R, int k) {
        const Image g = R.ring[k];
        const float *s = R.T.s + g.c * L_ES;
        const float c = s[T_C], rs = s[T_RS], cn = s[T_CN], rn = s[T_RN], mv = s[T_MV], mb = s[T_MOB],
                    un = R.T.s[(g.u >> 2) * L_ES + T_UN], vn = R.T.s[(g.v >> 2) * L_ES + T_VN];
        float *t = R.T.s + g.e * L_ES;
        t[T_C] = c; // (of the top level: the others' come with the restriction)
        t[T_RS] = rs;
        t[T_CN] = cn;
        t[T_RN] = rn;
        t[T_MV] = mv;
        t[T_MOB] = mb;
        t[T_UN] = signed_val((g.u & 3) - 1, un);
        t[T_VN] = signed_val((g.v & 3) - 1, vn);
        t[T_U] = t[T_U2] = t[T_V] = t[T_V2] = 0.0f; // on the faces of a high wall
    });
    __syncthreads();
    for (int p = 0; p < 2 * depth - 1; p++) {
        const int l = p < depth ? p : 2 * depth - 2 - p;
        const BotLevF B = bot_lev(smf, m1, m2, l);
        if (p > 0 && p < depth) bot_restrict(P, (&d)[l - 1], bot_lev(smf, m1, m2, l - 1), B);
        if (p >= depth) bot_prolong(P, d, B, bot_lev(smf, m1, m2, l + 1));
        const bool last = p == depth - 1;
        bot_smooth(P, (&d)[l], B, last ? nuc : p < depth ? nu1 : nu2, last ? comega : omega);
    }
    const BotLevF B = bot_lev(smf, m1, m2, 0);
    for (int e = threadIdx.x; e < m1 * m2; e += BOT) {
        const int j = e / m1, i = e - j * m1;
        const size_t q = (size_t)j * L.pitch + i;
        const float *t = B.T.at(i, j);
        sta<1>(L.dc, q, t[L_DC]);
        sta<1>(L.dmu, q, t[T_MU]);
        sta<1>(L.dp, q, t[T_P]);
        sta<1>(ua, q, t[T_U]);
        sta<1>(va, q, t[T_V]);
    }
}
QN_KERNEL(k_mx_bottom, __launch_bounds__(BOT), (int nu1, int nu2, int nuc, float omega, float comega), (nu1, nu2, nuc, omega, comega))

// w += delta on the finest level (FP64 state, single u/v buffer in mixed
// mode); faces on walls are not unknowns
template <typename IT> __device__ __forceinline__ void k_mx_update_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= d.m1 * d.m2) return;
    const int j = t / d.m1, i = t - j * d.m1;
    const size_t q = (size_t)j * d.pitch + i;
    const int par = it_par(it, k);
    d.c[q] += (double)d.dc[q];
    d.mu[q] += (double)d.dmu[q];
    d.p[q] += (double)d.dp[q];
    if (d.bcx || i >= 1) d.ub[0][q] += (double)d.dub[par][q];
    if (d.bcy || j >= 1) d.vb[0][q] += (double)d.dvb[par][q];
}
QN_KERNEL(k_mx_update, __launch_bounds__(BLK), (), ())

// FP32 time-n data of the next coarser level
template <typename IT> __device__ __forceinline__ void k_mx_restrict_n_body(const IT &it)
{
    const int k = find_item(it);
    const Desc &F = it_desc(it, k);
    const Desc &C = (&F)[1];
    const int t = ((int)blockIdx.x - it_start(it, k)) * BLK + threadIdx.x;
    if (t >= C.m1 * C.m2) return;
    const int J = t / C.m1, I = t - J * C.m1;
    const size_t f = (size_t)(2 * J) * F.pitch + 2 * I, q = (size_t)J * C.pitch + I;
    C.cnf[q] = 0.25f * (F.cnf[f] + F.cnf[f + 1] + F.cnf[f + F.pitch] + F.cnf[f + F.pitch + 1]);
    C.unf[q] = 0.5f * (F.unf[f] + F.unf[f + F.pitch]);
    C.vnf[q] = 0.5f * (F.vnf[f] + F.vnf[f + 1]);
}
QN_KERNEL(k_mx_restrict_n, __launch_bounds__(BLK), (), ())

// r - J delta on a level into the FP64 residual-field buffer (m1 x m2 per
// field, packed), for checking the linearisation
template <typename IT> __device__ __forceinline__ void k_mx_linresid_body(const IT &it)
{
    TILE_LDS float sm[L_ES * TILE_S * (TY + 2)];
    const int k = find_item(it);
    const Desc &d = it_desc(it, k);
    if (!tile_valid(it, k, d)) return;
    const LView L = lview_of(d, it_par(it, k));
    const TileF T = item_tile<TileF, TX + 2>(sm, it, k, d);
    ltile_load<2, TBLK>(d.Pf, L, T);
    __syncthreads();
    const size_t n = (size_t)L.m1 * L.m2;
    const int i = T.i0 + (int)threadIdx.x % TX, j = T.j0 + (int)threadIdx.x / TX;
    if (i >= L.m1 || j >= L.m2) return;
    const ResidF r = lresid_cell(d.Kf, L, T, i, j);
    const size_t q = (size_t)j * L.m1 + i;
    d.rout[q] = r.c;
    d.rout[n + q] = r.mu;
    d.rout[2 * n + q] = r.p;
    d.rout[3 * n + q] = r.u;
    d.rout[4 * n + q] = r.v;
}
QN_KERNEL(k_mx_linresid, __launch_bounds__(TBLK), (), ())

} // namespace qn
