// qnsch_lin.hpp -- FP32 linearised smoother of the mixed-precision step.
//
// Mixed precision solves the nonlinear system N(w) = 0 of sec. 6.1 by defect
// correction: the residual r = -N(w) and the update w += delta are FP64, and
// delta comes from one multigrid V-cycle on the linearisation
//     J(w^) delta = r,   w^ = w rounded to FP32,
// run entirely in FP32.  J is the exact Jacobian of the discrete equations
// (the same equations as the FP64 smoother, differentiated by hand), so the
// outer iteration is an inexact Newton method whose inner solve has the
// colour ordering, box smoother and transfers of the FP64 V-cycle (sec. 7.1).
//
// Nonlinear terms of N and their linearisations (rho* = rho(c), rho' =
// -alpha rho^2; every other coefficient is time-n data and constant):
//   phase    rho*(c)(c - c^n)/dt                     -> Jcc dc (pointwise)
//   chem.    rho* mubar, the bulk terms in c          -> pointwise in dc, dmu
//            |grad c|^2 r(c)                          -> 5-point in dc
//            div(A rho* grad c) (App. A.6)            -> 5-point in dc
//   momentum (A rho* - A rho^n) u/(2 dt)              -> faces: du, and dc of
//                                                        the two adjacent cells
// The rest (advection with time-n velocity, viscous, pressure, surface-tension
// and mass-equation terms) is linear in the unknowns and is applied to delta
// with the FP64 formulas; gravity and time-n sources drop out.
//
// Tile layout: the element of the FP64 tile (T_C holds c^, the linearisation
// point; T_MU, T_P, T_U, T_V the corrections dmu, dp, du, dv) with the
// correction dc and the induced change of density rho'(c^) dc behind it, so
// that the axis descriptor, the momentum rows and the box solve are shared.
#pragma once
#include "qnsch_dev.hpp"

namespace qn {

struct PhysF {
    float rho1, rho12, drho, visc1, visc12, dvisc;
    float alpha, mob_reg;
    int coupled; // smoother as in Phys
};

// one level of the correction problem
struct LView {
    const float *c, *mu, *u, *v;          // linearisation point (cells; faces)
    float *dc, *dmu, *dp;                 // correction of the cell unknowns
    const float *du, *dv;                 // correction of the faces (buffer being read)
    const float *cn, *un, *vn;            // time-n data
    const float *rc, *rmu, *rp, *ru, *rv; // right-hand side
    int m1, m2, pitch, bcx, bcy;
};

typedef TileT<float, L_ES> TileF;

__device__ __forceinline__ float frcpf(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rhof(const PhysF &P, float c) { return P.rho12 * frcpf(P.drho * c + P.rho1); }
__device__ __forceinline__ float viscf(const PhysF &P, float c) { return P.visc12 * frcpf(P.dvisc * c + P.visc1); }
__device__ __forceinline__ float mobf(const PhysF &P, float c)
{
    const float q = c * (1.0f - c);
    return __builtin_sqrtf(q * q + P.mob_reg);
}

// an element's fields from its nine loaded values (c^, dc, dmu, dp, du, dv,
// c^n, u^n, v^n) and the signs of its faces
__device__ __forceinline__ void ltile_put(const PhysF &P, float *t, int su, int sv, const float (&v)[9])
{
    const float rs = rhof(P, v[0]);
    t[T_C] = v[0];
    t[T_CN] = v[6];
    t[T_MU] = v[2];
    t[T_P] = v[3];
    t[T_RN] = rhof(P, v[6]);
    t[T_MV] = viscf(P, v[6]);
    t[T_RS] = rs;
    t[T_MOB] = mobf(P, v[6]);
    t[T_U] = signed_val(su, v[4]);
    t[T_UN] = signed_val(su, v[7]);
    t[T_V] = signed_val(sv, v[5]);
    t[T_VN] = signed_val(sv, v[8]);
    t[L_DC] = v[1];
    t[L_DRS] = -P.alpha * rs * rs * v[1];
}

// cooperative load of a tile, NE elements per thread (as tile_load)
template <int NE, int NT> __device__ __forceinline__ void ltile_load(const PhysF &P, const LView &L, const TileF &T)
{
    const int n = T.W * T.H;
    float v[NE][9];
    if (tile_inner(L.m1, L.m2, T.i0, T.j0, T.W, T.H)) {
#pragma unroll
        for (int k = 0; k < NE; k++) {
            const int e = min((int)threadIdx.x + k * NT, n - 1), b = e / T.W, a = e - b * T.W;
            const size_t q = (size_t)((T.j0 - 1 + b) * L.pitch + (T.i0 - 1 + a));
            const float *src[9] = { L.c, L.dc, L.dmu, L.dp, L.du, L.dv, L.cn, L.un, L.vn };
#pragma unroll
            for (int f = 0; f < 9; f++) v[k][f] = lda<1>(src[f], q);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < NE; k++) {
            const int e = threadIdx.x + k * NT, b = e / T.W, a = e - b * T.W;
            if (e < n) ltile_put(P, T.s + (b * T.S + a) * L_ES, 1, 1, v[k]);
        }
        return;
    }
    TileSrc s[NE];
#pragma unroll
    for (int k = 0; k < NE; k++) {
        const int e = min((int)threadIdx.x + k * NT, n - 1), b = e / T.W, a = e - b * T.W;
        s[k] = tile_src(L.m1, L.m2, L.pitch, L.bcx, L.bcy, T.i0 - 1 + a, T.j0 - 1 + b);
        const float w[9] = { lda<1>(L.c, s[k].c), lda<1>(L.dc, s[k].c), lda<1>(L.dmu, s[k].c), lda<1>(L.dp, s[k].c),
                             lda<1>(L.du, s[k].u), lda<1>(L.dv, s[k].v), lda<1>(L.cn, s[k].c), lda<1>(L.un, s[k].u),
                             lda<1>(L.vn, s[k].v) };
#pragma unroll
        for (int f = 0; f < 9; f++) v[k][f] = w[f];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < NE; k++) {
        const int e = threadIdx.x + k * NT, b = e / T.W, a = e - b * T.W;
        if (e >= n) continue;
        if (s[k].sc == 0) tile_zero(T, b * T.S + a);
        else ltile_put(P, T.s + (b * T.S + a) * L_ES, s[k].su, s[k].sv, v[k]);
    }
}

// one axis of the linearised cell equations at element s: as axis_cell on the
// corrections, with lr the linearised gradient-energy and capillary terms of
// the chemical row beside the pointwise ones (across a wall the mirrored
// ghost makes both the difference of c^ and that of dc vanish)
template <int ES>
__device__ __forceinline__ CellSum<float> laxis_cell(const Kon<float> &K, const float *s, const Ax<ES> &a, float r,
                                                     float drs)
{
    const bool wP = a.per || a.ia < a.ma - 1, wM = a.per || a.ia > 0;
    const float *sP = el<ES>(s, a.dn), *sM = el<ES>(s, -a.dn);
    const float mP = sP[T_MOB] + s[T_MOB], mM = sM[T_MOB] + s[T_MOB];
    const float S = s[T_MU] + K.alpha * s[T_P];
    const float fP = (sP[T_MU] + K.alpha * sP[T_P]) - S, fM = S - (sM[T_MU] + K.alpha * sM[T_P]);
    const float flux = mP * fP - mM * fM;
    const float gP = sP[T_CN] - s[T_CN], gM = s[T_CN] - sM[T_CN], dP = sP[T_C] - s[T_C], dM = s[T_C] - sM[T_C];
    const float eP = sP[L_DC] - s[L_DC], eM = s[L_DC] - sM[L_DC];
    const float uP = sP[a.fn], u0 = s[a.fn];
    CellSum<float> x;
    const float adv = (sP[T_RN] * gP) * uP + (sM[T_RN] * gM) * u0;
    x.s1 = K.hih * adv - K.km * flux;
    x.s2 = K.ih * (uP - u0) - K.akm * flux;
    x.sm = K.km * ((wP ? mP : 0.0f) + (wM ? mM : 0.0f));
    x.g = (dP * dP + dM * dM) + (gP * gP + gM * gM);
    const float hP = dP + gP, hM = dM + gM;
    const float R0 = s[T_RS] + s[T_RN];
    const float RP = (sP[T_RS] + sP[T_RN]) + R0, RM = (sM[T_RS] + sM[T_RN]) + R0;
    const float dL = ((sP[L_DRS] + s[L_DRS]) * hP - (sM[L_DRS] + s[L_DRS]) * hM) + (RP * eP - RM * eM);
    const float k2 = 2.0f * K.kg * r;
    x.lr = K.kl * dL - k2 * (dP * eP + dM * eM);
    const float w = (wP ? RP : 0.0f) + (wM ? RM : 0.0f);
    x.j = K.kl * (drs * (hP - hM) - w) - k2 * (dM - dP);
    return x;
}

// J delta for the three cell equations and the local 2x2 Jacobian in
// (c_ij, mubar_ij) at c^ (the matrix of the FP64 point smoother)
struct LCellEq {
    float Nc, Nmu, Np;
    float Jcc, Jcm, Jmc, Jmm;
};
__device__ __forceinline__ void lcell_r(const Kon<float> &K, const float *s, float &r, float &drs)
{
    const float t = -K.alpha * s[T_RS];
    r = t * s[T_RN];
    drs = t * s[T_RS];
}
__device__ __forceinline__ LCellEq lcell_eq(const Kon<float> &K, const float *s, const CellSum<float> &x, float r,
                                            float drs, float muh)
{
    const float c = s[T_C], n = s[T_CN], rs = s[T_RS], rn = s[T_RN], dc = s[L_DC], dmu = s[T_MU];
    LCellEq q;
    q.Jcc = K.idt * (drs * (c - n) + rs);
    q.Nc = q.Jcc * dc + x.s1;
    q.Np = x.s2;
    const float rh = 0.5f * (rs + rn);
    const float q1 = c * (c - 1.0f), q0 = n * (n - 1.0f), t = c + n - 1.0f, qs = q1 + q0;
    const float g = 0.25f * qs * t;
    const float Fh = 0.125f * (q1 * q1 + q0 * q0);
    const float G = K.kg * x.g + K.K1 * Fh;
    const float dg = 0.25f * ((2.0f * c - 1.0f) * t + qs);
    const float f1 = q1 * (c - 0.5f);
    const float dr = -K.alpha * rs * r;
    // derivative in the cell's own c of every term that is pointwise in it
    const float Jpw = drs * muh - K.K1 * (0.5f * (drs * g + f1 * r) + rh * dg) - G * dr;
    q.Nmu = rs * dmu + Jpw * dc + x.lr;
    q.Jcm = x.sm;
    q.Jmm = rs;
    q.Jmc = Jpw + x.j;
    return q;
}

// one cell of the current colour: the FP64 smoother applied to the
// correction equation J(w^) delta = r.  Segregated: step 1 is a 2x2 solve for
// (dc, dmu) of the cell, step 2 the 5x5 Vanka box for its four faces and dp.
// Coupled: the seven-unknown box of the FP64 smoother with the entries of J at
// w^ (the face rows' dc entry multiplies the face velocity at w^), solved the
// same way.
// With TO set, as relax_cell: the cell at tile position (ti, tj), results
// kept in the tile (dc, dmu, dp and the density change in place, the face
// corrections in the fields T_U2, T_V2).
template <int TO, int AS, bool HOOD>
__device__ __forceinline__ void lrelax_cell(const PhysF &P, const Kon<float> &K, const LView &L, const TileF &T,
                                            float *dunew, float *dvnew, int i, int j, int ti, int tj, int hlf,
                                            float omega, int slot = 0)
{
    constexpr int ES = TileF::ES;
    const CellPos<ES> b = cell_pos(L, T, i, j, hlf, slot);
    float *const e = T.at(ti, tj); // results go here, everything is read at s
    Hood<TileF, float> H;
    const float *s = e;
    Ax<ES> a = b.a;
    const bool cpl = P.coupled;
    const float muh = lda<AS>(L.mu, b.k), f_c = lda<AS>(L.rc, b.k), f_mu = lda<AS>(L.rmu, b.k),
                f_p = lda<AS>(L.rp, b.k);
    // the velocity at w^ and the right-hand sides on the lane's two faces
    // (west and east, or south and north, of the cell)
    const float *fw = hlf ? L.v : L.u, *fN = hlf ? L.rv : L.ru;
    const float uhlo = lda<AS>(fw, b.k), uhhi = lda<AS>(fw, b.khi);
    const float f_lo = lda<AS>(fN, b.k), f_hi = lda<AS>(fN, b.khi);
    if (HOOD) {
        a = H.template load<true, TO == 2>(e, b.a);
        s = H.centre();
    }
    float r, drs;
    lcell_r(K, s, r, drs);
    const CellSum<float> xo = laxis_cell(K, s, a, r, drs), x = xo + other(xo);
    const LCellEq q = lcell_eq(K, s, x, r, drs, muh);
    const float r1 = f_c - q.Nc, r2 = f_mu - q.Nmu;
    const float c0 = s[L_DC], m0 = s[T_MU], p0 = s[T_P], rs = s[T_RS];
    const float Jcp = K.alpha * x.sm;
    float bp = f_p - q.Np;
    float kmc = 0.0f, kbm = 0.0f, Jc = 0.0f, bc = 0.0f, gc = 0.0f;
    if (cpl) {
        const float imm = frcpf(q.Jmm);
        kmc = q.Jmc * imm;
        kbm = r2 * imm;
        Jc = q.Jcc - q.Jcm * kmc;
        bc = r1 - q.Jcm * kbm;
        gc = 0.5f * K.hidt * drs;
    } else {
        // ---- step 1
        const float idet = frcpf(q.Jcc * q.Jmm - q.Jcm * q.Jmc);
        const float cnew = c0 + (q.Jmm * r1 - q.Jcm * r2) * idet;
        const float dm = (q.Jcc * r2 - q.Jmc * r1) * idet, mnew = m0 + dm;
        if (!TO && hlf == 0) {
            sta<AS>(L.dc, b.k, cnew);
            sta<AS>(L.dmu, b.k, mnew);
        }
        const float drnew = -P.alpha * rs * rs * cnew;
        if (HOOD) {
            float *o = H.centre();
            o[L_DC] = cnew;
            o[T_MU] = mnew;
            o[L_DRS] = drnew;
        }
        if (TO || !HOOD) {
            e[L_DC] = cnew;
            e[T_MU] = mnew;
            e[L_DRS] = drnew;
        }
        bp -= Jcp * dm;
    }
    // ---- the box
    const FaceEq<float> flo = face_eq<float, false, true>(K, s, a, uhlo), fhi = face_eq<float, false, true>(K, el<ES>(s, a.dn), a, uhhi);
    const float *P1 = el<ES>(s, a.dn), *M1 = el<ES>(s, -a.dn);
    const float alo = b.hlo ? K.hih * (M1[T_RN] * (s[T_CN] - M1[T_CN])) : 0.0f;
    const float ahi = b.hhi ? K.hih * (P1[T_RN] * (P1[T_CN] - s[T_CN])) : 0.0f;
    float alh, ahl;
    box_offdiag(K, s, a, b.hlo, b.hhi, alh, ahl);
    const float sb = kbm * K.iM, sc = kmc * K.iM;
    const float blo = b.hlo ? (f_lo - flo.N) + sb * alo : 0.0f, bhi = b.hhi ? (f_hi - fhi.N) + sb * ahi : 0.0f;
    const float qlo = b.hlo ? gc * uhlo + sc * alo : 0.0f, qhi = b.hhi ? gc * uhhi + sc * ahi : 0.0f;
    const BoxAx<float> X = box_axis(b.hlo ? flo.diag : 1.0f, b.hhi ? fhi.diag : 1.0f, alh, ahl, blo, bhi,
                                    b.hlo ? 1.0f : 0.0f, b.hhi ? -1.0f : 0.0f, qlo, qhi, alo, ahi);
    float dp, dc, t, tt;
    box_solve(X, box_other(X), cpl, K.kv * s[T_MV], K.kp, K.ih, K.alpha * Jcp, Jcp, kmc, kbm, Jc, bp, bc, dp, dc, t, tt);
    const float nlo = s[a.fn] + omega * ((X.xb[0] + t * X.xs[0]) - dc * X.xq[0]);
    const float nhi = P1[a.fn] + omega * ((X.xb[1] + t * X.xs[1]) - dc * X.xq[1]);
    const float np = p0 + omega * dp;
    if (TO) {
        if (b.hlo) e[b.a.fo] = nlo;
        if (b.hhi) el<ES>(e, b.hi<TO>())[b.a.fo] = nhi;
        if (hlf == 0) {
            e[T_P] = np;
            if (cpl) {
                e[L_DC] = c0 + dc;
                e[T_MU] = m0 + (kbm - kmc * dc);
                e[L_DRS] = -P.alpha * rs * rs * (c0 + dc);
            }
        }
        return;
    }
    float *fo = hlf ? dvnew : dunew;
    if (b.hlo) sta<AS>(fo, b.k, nlo);
    if (b.hhi) sta<AS>(fo, b.khi, nhi);
    if (hlf == 0) {
        sta<AS>(L.dp, b.k, np);
        if (cpl) {
            sta<AS>(L.dc, b.k, c0 + dc);
            sta<AS>(L.dmu, b.k, m0 + (kbm - kmc * dc));
        }
    }
}

// residual of the correction equation r - J(w^) delta for the five equations
// attached to cell (i, j) (cell equations, west and south face, zero for a
// face on a wall), by one lane; the level is in global memory
struct ResidF {
    float c, mu, p, u, v;
};
template <int AS = 1>
__device__ __forceinline__ ResidF lresid_cell(const Kon<float> &K, const LView &L, const TileF &T, int i, int j)
{
    const size_t k = (size_t)j * L.pitch + i;
    const float *e = T.at(i, j);
    constexpr int ES = TileF::ES;
    const Ax<ES> ax = make_ax(L, T, i, j, 0), ay = make_ax(L, T, i, j, 1);
    const ResidF f = { lda<AS>(L.rc, k), lda<AS>(L.rmu, k), lda<AS>(L.rp, k), lda<AS>(L.ru, k), lda<AS>(L.rv, k) };
    const float muh = lda<AS>(L.mu, k), uh = lda<AS>(L.u, k), vh = lda<AS>(L.v, k);
    float r, drs;
    lcell_r(K, e, r, drs);
    const CellSum<float> x = laxis_cell(K, e, ax, r, drs) + laxis_cell(K, e, ay, r, drs);
    const LCellEq q = lcell_eq(K, e, x, r, drs, muh);
    const FaceEq<float> fu = face_eq<float, false, true>(K, e, ax, uh), fv = face_eq<float, false, true>(K, e, ay, vh);
    return { f.c - q.Nc, f.mu - q.Nmu, f.p - q.Np, ax.per || i >= 1 ? f.u - fu.N : 0.0f,
             ay.per || j >= 1 ? f.v - fv.N : 0.0f };
}

} // namespace qn
