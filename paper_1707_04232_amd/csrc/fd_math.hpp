// Device math of one fluctuation/dissipation pair update (Sec. 3.2-3.3 of
// Faure & Stoltz): Philox4x32-10 draws, the Ornstein-Uhlenbeck proposal in
// the relative velocity, the energy bound and the Metropolis log-ratio.
#pragma once

#include "sdpd_internal.hpp"
#include "fd_elem.hpp"

namespace sdpd {

// ---------------------------------------------------------------- constants
// The polynomial coefficients of the draws and of the pair update, as scalar
// loads at the place that uses them.  Written as literals they are moved out of
// the persistent loop of the sweep and held in registers for the whole kernel;
// some 100 of them displaced what the level steps need (spills into vector
// lanes, parameters read from memory inside the loop).  `cold` keeps the loads
// below the point where it is called.
typedef const __attribute__((address_space(4))) double ColdTable;
__device__ __forceinline__ ColdTable *cold(const double *tab)
{
    ColdTable *c = (ColdTable *)tab;
    __asm__ volatile("" : "+s"(c));
    return c;
}

static __constant__ double kExpm1Tab[15] = {SDPD_EXPM1_COEF};
static __constant__ double kLogTab[14] = {SDPD_LOG_COEF};
constexpr int kDrawSinCos = 14;   // draws: the log table, then sine and cosine
static __constant__ double kDrawTab[34] = {SDPD_LOG_COEF, SDPD_SINCOS_COEF};

// expm1 of the friction exponents
__device__ __forceinline__ double expm1_wave(double x, ColdTable *t)
{
    return elem_expm1_wave(x, t, [] { return cold(kExpm1Tab); });
}

// ---------------------------------------------------------------- Philox
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each two
// 32x32->64 products with multipliers 0xD2511F53 and 0xCD9E8D57, key
// advanced by the Weyl constants 0x9E3779B9 and 0xBB67AE85 between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t &x0, uint32_t &x1, uint32_t &x2,
                                              uint32_t &x3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t a = (uint64_t)0xD2511F53u * x0;
        const uint64_t b = (uint64_t)0xCD9E8D57u * x2;
        const uint32_t y0 = (uint32_t)(b >> 32) ^ x1 ^ k0;
        const uint32_t y2 = (uint32_t)(a >> 32) ^ x3 ^ k1;
        x1 = (uint32_t)b;
        x3 = (uint32_t)a;
        x0 = y0;
        x2 = y2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

__device__ __forceinline__ double open_unit(uint32_t w)
{
    return fma((double)w, 0x1p-32, 0x1p-33);   // (w + 1/2) 2^-32, exact
}

// Gaussian vector (Box-Muller on the first block) and the word of the uniform
// U = open_unit(u) of one pair
__device__ __forceinline__ void pair_draws(const DevParams &P, uint32_t step, uint32_t id_i,
                                           uint32_t id_j, double G[3], uint32_t &u, ColdTable *t)
{
#pragma clang fp contract(fast)
    uint32_t a0 = step, a1 = id_i, a2 = id_j, a3 = P.replica * 2u;
    uint32_t b0 = step, b1 = id_i, b2 = id_j, b3 = P.replica * 2u + 1u;
    philox4x32_10(a0, a1, a2, a3, P.seed_lo, P.seed_hi);
    philox4x32_10(b0, b1, b2, b3, P.seed_lo, P.seed_hi);
    const double R1 = fd_sqrt(-2.0 * elem_log(open_unit(a0), t));
    const double R2 = fd_sqrt(-2.0 * elem_log(open_unit(a2), t));
    double s1, c1;
    elem_sincospi(2.0 * open_unit(a1), s1, c1, t + kDrawSinCos);
    G[0] = R1 * c1;
    G[1] = R1 * s1;
    G[2] = R2 * elem_cospi(2.0 * open_unit(a3), t + kDrawSinCos);
    u = b0;
}

// Mixed precision: the Gaussian vector from the same Philox words through
// Box-Muller in FP32.  The radius sqrt(-2 ln u) takes ln u as log1p(-(1 - u))
// for u > 1/2, with 1 - u formed from the complement word, so that u near 1
// keeps its relative precision (log1p(x) = ln(1 + x) x / ((1 + x) - 1)
// compensates the rounding of 1 + x); the angles 2 pi t go to the hardware
// sine and cosine, whose argument is in turns.  U stays the FP64 uniform.
__device__ __forceinline__ float radius_f32(uint32_t w)
{
    const bool hi = w >= 0x80000000u;
    const float v = ((float)(hi ? ~w : w) + 0.5f) * 2.3283064365386963e-10f;   // u or 1 - u
    const float y = 1.0f - v;
    const float l1 = y == 1.0f ? -v : __logf(y) * (-v / (y - 1.0f));
    const float l = hi ? l1 : __logf(v);
    return sqrtf(-2.0f * l);
}
__device__ __forceinline__ float turns_f32(uint32_t w)
{
    return ((float)w + 0.5f) * 2.3283064365386963e-10f;
}
__device__ __forceinline__ void gauss3_f32(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3,
                                           double G[3])
{
    const float R1 = radius_f32(a0), R2 = radius_f32(a2);
    const float t1 = turns_f32(a1), t3 = turns_f32(a3);
    G[0] = (double)(R1 * __builtin_amdgcn_cosf(t1));
    G[1] = (double)(R1 * __builtin_amdgcn_sinf(t1));
    G[2] = (double)(R2 * __builtin_amdgcn_cosf(t3));
}
__device__ __forceinline__ void pair_draws_f32(const DevParams &P, uint32_t step, uint32_t id_i,
                                               uint32_t id_j, double G[3], uint32_t &u)
{
    uint32_t a0 = step, a1 = id_i, a2 = id_j, a3 = P.replica * 2u;
    uint32_t b0 = step, b1 = id_i, b2 = id_j, b3 = P.replica * 2u + 1u;
    philox4x32_10(a0, a1, a2, a3, P.seed_lo, P.seed_hi);
    philox4x32_10(b0, b1, b2, b3, P.seed_lo, P.seed_hi);
    gauss3_f32(a0, a1, a2, a3, G);
    u = b0;
}

// ---------------------------------------------------------------- coefficients
// alpha^theta and the squared relative-velocity noise amplitude
// b^theta^2 = ((2/m) zeta^theta)^2 at energies (ei, ej).  With
// gamma = kappa (1 - d) and sigma^2 = 4 kappa kB T_i T_j/(T_i + T_j) of
// eq. (sdpd-gamma-sigma), zeta^2 = sigma^2 m (1 - alpha^2)/(4 gamma) reduces
// to m kB T_red (1 - alpha^2)/(1 - d) with T_red = T_i T_j/(T_i + T_j), so
// b^2 = (4 kB/m) T_red (1 - alpha^2)/(1 - d).  With e = expm1(-2 gamma dt/m):
// alpha = 1 + e and 1 - alpha^2 = -e (2 + e), both without cancellation.
// The constants of the pair update, held in vector registers by the level loop
// (read once per batch): read from the parameters inside the loop they become
// vector loads there, whose waits also hold up the prefetch of the records.
template <bool MIX>
struct PairRegs {
    double inv_m, m_over_8, m_over_2, ent_c, d_c, b2_red;
    ColdTable *tab;   // expm1
    __device__ __forceinline__ PairRegs(const DevParams &P)
        : inv_m(P.inv_m), m_over_8(P.m_over_8), m_over_2(P.m_over_2), ent_c(P.ent_c),
          d_c(P.d_c), b2_red(P.b2_red), tab(cold(kExpm1Tab))
    {
        __asm__ volatile("" : "+v"(inv_m), "+v"(m_over_8), "+v"(m_over_2), "+v"(ent_c));
        if (!MIX) __asm__ volatile("" : "+v"(d_c), "+v"(b2_red));
    }
};

struct Coef {
    double e_par, e_perp;   // alpha - 1
    double q_par, q_perp;   // alpha^2 - 1 = e (2 + e)
    double b2_par, b2_perp;
    double b_par, b_perp;   // square roots of b2 (set by fd_coef_f32 only)
};

// At energies of sum S and product Q (T_red = Q / (Cv S), d = (2 kB/Cv) Q/S^2)
// and the pair's exponent y = -2 dt kappa_perp / m (that of d = 0).  When
// zeta = 0 the parallel friction is exactly twice the perpendicular one, and
// expm1(2x) = e (2 + e) with e = expm1(x) saves one exponential (and is also
// q_perp).  FAST = the common case fixed at compile time: EMS, Lucy, zeta = 0
template <bool FAST>
__device__ __forceinline__ Coef fd_coef(const DevParams &P, const PairRegs<false> &c, double y, double S,
                                        double Q)
{
#pragma clang fp contract(fast)
    const double inv_S = fast_rcp(S);
    const double red = Q * inv_S;
    const double omd = 1.0 - c.d_c * (red * inv_S);
    const double ye = y * omd;
    Coef r;
    r.e_perp = expm1_wave(ye, c.tab);
    r.q_perp = r.e_perp * (2.0 + r.e_perp);
    r.e_par = (FAST || P.par_twice_perp) ? r.q_perp : expm1_wave(ye * P.kpar_over_kperp, c.tab);
    r.q_par = r.e_par * (2.0 + r.e_par);
    const double s = c.b2_red * red * fast_rcp(omd);
    r.b2_par = -s * r.q_par;
    r.b2_perp = -s * r.q_perp;
    return r;
}

// ---------------------------------------------------------------- FP32 proposal
// Mixed precision: the geometry and the proposal coefficients e = alpha - 1
// and b of eq. (proposal) in FP32 (hardware reciprocal, square root and
// exponential), for the forward and the reverse move alike.  The proposal
// v' = alpha v + b G, the energies, Delta and the Metropolis log-ratio of
// eq. (metropolis-ratio) stay FP64 and use exactly these coefficients: alpha
// = 1 + e and b are FP32 values promoted, b^2 is formed in FP64 from b (an
// exact square), so the ratio is the exact one of the FP32-defined proposal.

// expm1(x): Taylor polynomial to x^8 for |x| < 1/2 (its tail is below
// 2^-26 |x| there), exp(x) - 1 otherwise (no cancellation for |x| >= 1/2)
__device__ __forceinline__ float expm1_f32(float x)
{
    float p = 2.4801587e-05f;        // 1/8!
    p = fmaf(p, x, 1.9841270e-04f);  // 1/7!
    p = fmaf(p, x, 1.3888889e-03f);  // 1/6!
    p = fmaf(p, x, 8.3333333e-03f);  // 1/5!
    p = fmaf(p, x, 4.1666668e-02f);  // 1/4!
    p = fmaf(p, x, 1.6666667e-01f);  // 1/3!
    p = fmaf(p, x, 0.5f);
    const float small = fmaf(p * x, x, x);
    const float big = __expf(x) - 1.0f;
    return fabsf(x) < 0.5f ? small : big;
}

// the coefficients at energies (ei, ej), EMS with Lucy's kernel and zeta = 0
// (kpar = 2 kperp, so e_par = e_perp (2 + e_perp)); kperp in FP32
__device__ __forceinline__ Coef fd_coef_f32(const DevParams &P, float kperp, double ei, double ej,
                                            float dt)
{
    const float Ti = (float)ei * P.inv_Cv_f, Tj = (float)ej * P.inv_Cv_f;
    const float inv_Ts = __builtin_amdgcn_rcpf(Ti + Tj);
    const float Tred = Ti * Tj * inv_Ts;
    const float d = P.d_c_f * Tred * inv_Ts;
    const float omd = 1.0f - d;
    const float c = -2.0f * dt * P.inv_m_f * omd;
    const float e_perp = expm1_f32(c * kperp);
    const float e_par = e_perp * (2.0f + e_perp);
    const float s = P.b2_c_f * Tred * __builtin_amdgcn_rcpf(omd);
    const float bp = __builtin_amdgcn_sqrtf(-s * e_par * (2.0f + e_par));
    const float bq = __builtin_amdgcn_sqrtf(-s * e_perp * (2.0f + e_perp));
    Coef r;
    r.e_par = (double)e_par;
    r.e_perp = (double)e_perp;
    r.q_par = fma(r.e_par, r.e_par, 2.0 * r.e_par);
    r.q_perp = fma(r.e_perp, r.e_perp, 2.0 * r.e_perp);
    r.b_par = (double)bp;
    r.b_perp = (double)bq;
    r.b2_par = r.b_par * r.b_par;
    r.b2_perp = r.b_perp * r.b_perp;
    return r;
}

struct FdCount {
    uint32_t proposed, rej_energy, rej_ratio, marginal, negeps;
};

// Everything of one oriented pair (i = smaller id) that does not change
// during a sweep: the unit vector e_ij, the exponent y = -2 dt kappa_perp/m
// (mixed precision: kappa_perp itself, an FP32 value), the Gaussian vector,
// the Philox word of the uniform and the pair's two places in the batch (i in
// the low half).  Formed once per pair at full lane occupancy before the level
// steps, where lanes idle: 64 bytes a pair, stored as four planes of 16 bytes
// so that the lanes of a step read consecutive addresses.
struct PairRec {
    double ex, ey, ez, y, G0, G1, G2;
    uint32_t u, ij;
};

// separation component d = x_i - x_j to its minimum image: the same rounding
// as adding the shift -+box where |d| > box/2 (k box is exact for |k| <= 1)
__device__ __forceinline__ double nearest_image(double d, double box, double inv_box)
{
    return fma(-rint(d * inv_box), box, d);
}

// K: 0 = general, 1 = EMS, Lucy, zeta = 0, 2 = that case with the FP32 proposal
template <int K>
__device__ __forceinline__ PairRec pair_record(const DevParams &P, double y_c, uint32_t step,
                                               uint32_t id_i, uint32_t id_j, double4 a, double4 b,
                                               ColdTable *t)
{
#pragma clang fp contract(fast)
    // geometry (Sec. 2.1.1): r_ij, e_ij, F_ij
    const double dx = nearest_image(a.x - b.x, P.box[0], P.inv_box[0]);
    const double dy = nearest_image(a.y - b.y, P.box[1], P.inv_box[1]);
    const double dz = nearest_image(a.z - b.z, P.box[2], P.inv_box[2]);
    PairRec r;
    if (K == 2) {
        const float xf = (float)dx, yf = (float)dy, zf = (float)dz;
        const float r2 = xf * xf + yf * yf + zf * zf;
        const float inv_r = __builtin_amdgcn_rsqf(r2);
        const float w = 1.0f - r2 * inv_r * P.inv_h_f;
        r.ex = (double)(xf * inv_r);
        r.ey = (double)(yf * inv_r);
        r.ez = (double)(zf * inv_r);
        // kappa_perp of Sec. 2.2.2 with Lucy's F
        r.y = (double)(P.kperp_c_f * (P.cF_f * (w * w)) *
                       __builtin_amdgcn_rcpf((float)(a.w * b.w)));
    } else {
        const double r2 = dx * dx + dy * dy + dz * dz;
        const double inv_r = fast_rsq(r2);
        r.ex = dx * inv_r;
        r.ey = dy * inv_r;
        r.ez = dz * inv_r;
        const double x = r2 * inv_r * P.inv_h, w = 1.0 - x;
        double F;   // over its prefactor cF, which y_c holds
        if (K == 1 || P.kernel == SDPD_KERNEL_LUCY) F = w * w;
        else F = x <= 0.5 ? 2.0 - 3.0 * x : P.h * (w * w) * inv_r;
        r.y = y_c * F * fast_rcp(a.w * b.w);
    }
    double G[3];
    if (K == 2) pair_draws_f32(P, step, id_i, id_j, G, r.u);   // FP32 Box-Muller
    else pair_draws(P, step, id_i, id_j, G, r.u, t);
    r.G0 = G[0];
    r.G1 = G[1];
    r.G2 = G[2];
    return r;
}

// x - x^2/2 + x^3/3.  For |x| <= 1/2 the alternating series of log(1 + x)
// puts log(1 + x) within x^4/2 of it (the tail after the cubic term is at
// most |x|^4 / (4 (1 - |x|))).
__device__ __forceinline__ double log1p_cubic(double x)
{
    return x * fma(x, fma(x, 0.3333333333333333, -0.5), 1.0);
}

// Brackets closer than this are decided with the logarithms evaluated: it
// covers the 1e-9 window in which a decision counts as marginal plus the
// rounding of both evaluations (below 1e-13 for the values that occur).
constexpr double kLazyMargin = 2e-9;

// One pair update; the low half of g.ij has the smaller id.  The state of a particle is
// (p_x, p_y, p_z, eps) in LDS.  K as in pair_record.
//
// The move is written in scalars of the pair: with v_par = v.e, the
// perpendicular parts enter only through |v_perp|^2 = v^2 - v_par^2,
// v_perp.G_perp = v.G - v_par G_par and |G_perp|^2 = G^2 - G_par^2, and every
// difference is formed from e = alpha - 1, so that
//   |v'|^2 - |v|^2 = sum_theta q |v|^2 + 2 alpha b (v.G) + b^2 |G|^2,
//   v - alpha' v'  = -(E v + alpha' b G),  E = e + e' + e e' = alpha alpha' - 1
// have no cancelling terms of order v^2 (the reverse move's quadratic form is
// of order b^2).
template <int K>
__device__ __forceinline__ void fd_pair(const DevParams &P, const PairRegs<K == 2> &c, double dt,
                                        const PairRec &g, double2 *s_st, FdCount &cnt,
                                        bool &negeps)
{
#pragma clang fp contract(fast)
    constexpr bool FAST = K != 0, MIX = K == 2;
    const uint32_t li = g.ij & 0xFFFFu, lj = g.ij >> 16;
    const double2 i0 = s_st[2 * li], i1 = s_st[2 * li + 1];
    const double2 j0 = s_st[2 * lj], j1 = s_st[2 * lj + 1];
    const double px = i0.x - j0.x, py = i0.y - j0.y, pz = i1.x - j1.x;
    const double ei = i1.y, ej = j1.y;
    const double vpar = (px * g.ex + py * g.ey + pz * g.ez) * c.inv_m;
    const double vG = (px * g.G0 + py * g.G1 + pz * g.G2) * c.inv_m;
    const double v2 = (px * px + py * py + pz * pz) * (c.inv_m * c.inv_m);
    const double Gpar = g.G0 * g.ex + g.G1 * g.ey + g.G2 * g.ez;
    const double G2 = g.G0 * g.G0 + g.G1 * g.G1 + g.G2 * g.G2;
    const double vv = vpar * vpar, vg = vpar * Gpar, gg = Gpar * Gpar;
    // |v_perp|^2 = v^2 - (1 + z) v_par^2 with z = 1 - |e|^2, and so on: z is
    // rounding (taken as 0) unless e_ij is an FP32 vector
    const double z = MIX ? 1.0 - (g.ex * g.ex + g.ey * g.ey + g.ez * g.ez) : 0.0;
    const double z1 = 1.0 + z;
    const double vvq = MIX ? v2 - vv * z1 : v2 - vv;
    const double vgq = MIX ? vG - vg * z1 : vG - vg;
    const double ggq = MIX ? G2 - gg * z1 : G2 - gg;

    // proposal, eq. (proposal): v' = A(v) v + B(v) G, B = (2/m) zeta^theta P^theta
    const double S = ei + ej, Q = ei * ej;
    auto coef = [&](double a, double b, double sum, double product) -> Coef {
        if constexpr (MIX) return fd_coef_f32(P, (float)g.y, a, b, (float)dt);
        else return fd_coef<FAST>(P, c, g.y, sum, product);
    };
    const Coef f = coef(ei, ej, S, Q);
    const double b_par = MIX ? f.b_par : fd_sqrt(f.b2_par);
    const double b_perp = MIX ? f.b_perp : fd_sqrt(f.b2_perp);
    // energy change, eq. (proposal-update)
    const double ab_par = b_par + f.e_par * b_par, ab_perp = b_perp + f.e_perp * b_perp;
    double dv2 = (f.q_par * vv + (2.0 * ab_par) * vg + f.b2_par * gg) +
                 (f.q_perp * vvq + (2.0 * ab_perp) * vgq + f.b2_perp * ggq);
    if (MIX) {   // |e| != 1: the parts of v' along e and across it are not orthogonal
        const double n_par = vpar + (f.e_par * vpar + b_par * Gpar);
        const double n_perp = vpar + (f.e_perp * vpar + b_perp * Gpar);
        dv2 += z * (2.0 * n_par * n_perp - n_par * n_par - vv);
    }
    const double delta = c.m_over_8 * dv2;
    const double emin = fmin(ei, ej);
    bool accept = true;
    cnt.proposed += 1;
    if (!FAST && P.fd == SDPD_FD_SSA) {
        if (!(ei - delta > 0.0 && ej - delta > 0.0)) {
            cnt.negeps += 1;
            negeps = true;
        }
    } else {
        if (fabs(emin - delta) <= 1e-12 * fmax(fabs(emin), fabs(delta))) cnt.marginal += 1;
        if (!(emin > delta)) {                       // eq. (energy-bound)
            accept = false;
            cnt.rej_energy += 1;
        } else if (FAST || P.fd == SDPD_FD_EMS) {
            // reverse move from v' at the proposed energies, eq. (metropolis-ratio)
            const double ei2 = ei - delta, ej2 = ej - delta;
            const Coef r = coef(ei2, ej2, ei2 + ej2, ei2 * ej2);
            const double E_par = f.e_par + (r.e_par + f.e_par * r.e_par);
            const double E_perp = f.e_perp + (r.e_perp + f.e_perp * r.e_perp);
            const double c_par = b_par + r.e_par * b_par, c_perp = b_perp + r.e_perp * b_perp;
            const double w_par = E_par * vpar + c_par * Gpar;
            const double ww_perp =
                (E_perp * E_perp) * vvq + c_perp * ((2.0 * E_perp) * vgq + c_perp * ggq);
            // one reciprocal serves both inverse variances and the determinant
            // ratio, inv = 1/(b'_par^2 b'_perp^2), and the energies' 1/Q
            const double bb = r.b2_par * r.b2_perp, inv_all = fast_rcp(bb * Q);
            const double inv = inv_all * Q;
            const double quad = (w_par * w_par * r.b2_perp + ww_perp * r.b2_par) * inv;
            const double A = 0.5 * (G2 - quad);
            // log|B(v)| - log|B(v')| = (1/2) log Dr, Dr = b_par^2 b_perp^4 / (b'_par^2 b'_perp^4)
            const double Dr = (f.b2_par * f.b2_perp * f.b2_perp) * (r.b2_par * (inv * inv));
            // ideal gas: sum_k (S(eps'_k) - S(eps_k))/kB - log T(eps'_k) + log T(eps_k)
            //          = (Cv/kB - 1) log(1 + w), 1 + w = (1 - delta/ei)(1 - delta/ej)
            const double w = delta * (delta - S) * (inv_all * bb);
            const double U = open_unit(g.u);
            // a = A + logdet + ent is compared with log U (reject iff U > exp(a)).
            // Both are first bracketed with the cubic bounds of log1p_cubic;
            // the logarithms are evaluated only when the brackets come within
            // kLazyMargin of each other, which keeps every decision and the
            // marginal count equal to those of the evaluated comparison.
            bool evaluate = true;
            const double xd = Dr - 1.0, xu = U - 1.0;
            if (fabs(xd) <= 0.5 && fabs(w) <= 0.5) {
                const double xd2 = xd * xd, w2 = w * w;
                const double am = A + 0.5 * log1p_cubic(xd) + c.ent_c * log1p_cubic(w);
                const double ar = 0.25 * xd2 * xd2 + 0.5 * fabs(c.ent_c) * w2 * w2;
                double lu_lo, lu_hi;
                if (xu >= -0.5) {
                    const double xu2 = xu * xu;
                    const double um = log1p_cubic(xu);
                    lu_lo = um - 0.5 * xu2 * xu2;
                    lu_hi = um + 0.5 * xu2 * xu2;
                } else {   // U < 1/2: log U < log(1/2) < -0.69
                    lu_lo = -INFINITY;
                    lu_hi = -0.69;
                }
                if (lu_hi < am - ar - kLazyMargin) {
                    evaluate = false;                // log U < a: accept
                } else if (lu_lo > am + ar + kLazyMargin) {
                    evaluate = false;                // log U > a: reject
                    accept = false;
                    cnt.rej_ratio += 1;
                }
            }
            if (evaluate) {
                ColdTable *t = cold(kLogTab);
                const double logdet = 0.5 * elem_log(Dr, t);
                const double ent = c.ent_c * elem_log1p(w, t);
                const double a = A + logdet + ent;
                const double lnU = elem_log(U, t);
                if (fabs(a - lnU) <= 1e-9) cnt.marginal += 1;
                if (!(lnU <= a)) {
                    accept = false;
                    cnt.rej_ratio += 1;
                }
            }
        }
    }
    if (accept) {
        // dp = (m/2)(v' - v): along e, along v (in momentum units) and along G
        const double ke = c.m_over_2 * ((f.e_par - f.e_perp) * vpar + (b_par - b_perp) * Gpar);
        const double kp = 0.5 * f.e_perp, kg = c.m_over_2 * b_perp;
        const double dpx = ke * g.ex + (kp * px + kg * g.G0);
        const double dpy = ke * g.ey + (kp * py + kg * g.G1);
        const double dpz = ke * g.ez + (kp * pz + kg * g.G2);
        s_st[2 * li] = make_double2(i0.x + dpx, i0.y + dpy);
        s_st[2 * li + 1] = make_double2(i1.x + dpz, ei - delta);
        s_st[2 * lj] = make_double2(j0.x - dpx, j0.y - dpy);
        s_st[2 * lj + 1] = make_double2(j1.x - dpz, ej - delta);
    }
}

// ---------------------------------------------------------------- wave helpers
__device__ __forceinline__ uint64_t xor_permute_bits(uint64_t m, uint32_t x)
{
    // bit b of m moves to bit b ^ x
    const uint64_t M[6] = {0x5555555555555555ull, 0x3333333333333333ull,
                           0x0F0F0F0F0F0F0F0Full, 0x00FF00FF00FF00FFull,
                           0x0000FFFF0000FFFFull, 0x00000000FFFFFFFFull};
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int sh = 1 << k;
        const uint64_t sw = ((m & M[k]) << sh) | ((m >> sh) & M[k]);
        m = ((x >> k) & 1u) ? sw : m;
    }
    return m;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off);
    return v;
}

}  // namespace sdpd
