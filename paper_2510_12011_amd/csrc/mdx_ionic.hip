// Pointwise ionic-model kernels: one thread per mesh node, states stored
// structure-of-arrays (u[s * ld + i]) so every state load/store of a
// wavefront is one contiguous segment.
//
// The operator split of the paper's Eq. (2): states advance from (V^k, u^k)
// (gating variables by Rush-Larsen y <- y_inf + (y - y_inf) exp(-dt/tau),
// the other states by forward Euler), then the current is evaluated at
// (V^k, u^{k+1}).  Currents are per unit capacitance (pA/pF = mV/ms); the
// tissue's Cm (uF/mm^2) turns them into uA/mm^2.
//
// Models (the paper names them without equations; written from the original
// publications):
//  * Mitchell-Schaeffer two-variable model (Bull. Math. Biol. 2003), with the
//    membrane variable u = (V - v_rest) / v_amp and gate h;
//  * ten Tusscher-Panfilov 2006 human ventricular model, endocardial cell
//    (Am. J. Physiol. Heart Circ. Physiol. 291:H1088), 18 states + V;
//  * Courtemanche-Ramirez-Nattel 1998 human atrial model (Am. J. Physiol.
//    275:H301), 20 states + V.
#include "mdx_cellmath.h"
#include "mdx_device.h"
#include "mdx_internal.h"

namespace mdx {

namespace {

enum { MDX_KIND_NONE = 0, MDX_KIND_MS = 1, MDX_KIND_TT = 2, MDX_KIND_CRN = 3 };
constexpr int MS_NP = 7;
constexpr int TT_NS = 18;
constexpr int TT_NP = 12;

struct IonicParams {
    double v[16];
};

// Rush-Larsen step y <- y_inf + (y - y_inf) exp(-dt/tau).  In FP32 it is
// evaluated as y + (y_inf - y) (1 - exp(-dt/tau)) with expm1: exp(-dt/tau)
// is within 1e-4 of 1, and rounding it to FP32 would misstate the decay
// rate by ~1e-3, an error that accumulates step after step.
__device__ __forceinline__ double rush_larsen(double y, double y_inf, double tau, double dt)
{
    return y_inf - (y_inf - y) * exp(-dt / tau);
}
__device__ __forceinline__ float rush_larsen(float y, float y_inf, float tau, float dt)
{
    return y - (y_inf - y) * expm1f(-dt / tau);
}
// the same step given the rate 1/tau
__device__ __forceinline__ float rush_larsen_rate(float y, float y_inf, float rate, float dt)
{
    return y - (y_inf - y) * expm1f(-dt * rate);
}

// ---------------------------------------------------------------------------
// Mitchell-Schaeffer: params tau_in, tau_out, tau_open, tau_close, u_gate,
// v_rest, v_amp.  dh/dt = (1-h)/tau_open below u_gate, -h/tau_close above;
// I_ion/Cm = -v_amp (h u^2 (1-u)/tau_in - u/tau_out).
// ---------------------------------------------------------------------------
template <typename G>
__device__ __forceinline__ double ms_point(const IonicParams &P, double dt, double V, G &h)
{
    const double tau_in = P.v[0], tau_out = P.v[1], tau_open = P.v[2], tau_close = P.v[3];
    const double u_gate = P.v[4], v_rest = P.v[5], v_amp = P.v[6];
    double u = (V - v_rest) / v_amp;
    bool recovering = u < u_gate;
    G h_inf = recovering ? G(1) : G(0);
    G tau = (G)(recovering ? tau_open : tau_close);
    h = rush_larsen(h, h_inf, tau, (G)dt);
    return -v_amp * ((double)h * u * u * (1.0 - u) / tau_in - u / tau_out);
}

// ---------------------------------------------------------------------------
// ten Tusscher-Panfilov 2006, endocardial.
// State slots: Ki Nai Cai CaSR CaSS Rbar | xr1 xr2 xs m h j d f f2 fCass s r
// Params: GNa GK1 Gto GKr GKs GCaL GbNa GbCa GpCa GpK PNaK kNaCa
// ---------------------------------------------------------------------------
enum { KI, NAI, CAI, CASR, CASS, RBAR, XR1, XR2, XS, MG, HG, JG, DG, FG, F2G, FCASS, SG, RG };

// cell and environment constants
constexpr double Rgas = 8314.472, Temp = 310.0, Far = 96485.3415;
constexpr double RTONF = Rgas * Temp / Far;
constexpr double CAPAC = 0.185, VOLC = 0.016404, VOLSR = 0.001094, VOLSS = 0.00005468;
constexpr double K_O = 5.4, NA_O = 140.0, CA_O = 2.0;
constexpr double P_KNA = 0.03, KM_K = 1.0, KM_NA = 40.0, KM_NAI = 87.5, KM_CA = 1.38;
constexpr double K_SAT = 0.1, NCX_GAMMA = 0.35, NCX_ALPHA = 2.5, K_PCA = 0.0005;
constexpr double BUF_C = 0.2, KBUF_C = 0.001, BUF_SR = 10.0, KBUF_SR = 0.3;
constexpr double BUF_SS = 0.4, KBUF_SS = 0.00025;
constexpr double VMAX_UP = 0.006375, K_UP = 0.00025, V_REL = 0.102;
constexpr double K1_PRIME = 0.15, K2_PRIME = 0.045, K3 = 0.06, K4 = 0.005;
constexpr double EC_SR = 1.5, MAX_SR = 2.5, MIN_SR = 1.0;
constexpr double V_LEAK = 0.00036, V_XFER = 0.0038;

constexpr double TT_V_REST = -85.23;
__constant__ double TT_U0[TT_NS] = {136.89,   8.604,    0.000126, 3.64,   0.00036, 0.9073,
                                    0.00621,  0.4712,   0.0095,   0.00172, 0.7444, 0.7045,
                                    3.373e-5, 0.7888,   0.9755,   0.9953, 0.999998, 2.42e-8};

__device__ __forceinline__ double sq(double x) { return x * x; }

// factors of the currents that depend on V only
struct VOnly {
    double ical_drive;   // 2F * w/expm1(w) with w = 2(V-15)F/RT
    double ical_ew;      // exp(w) / 4
    double nak;          // pNaK K_o/(K_o + K_mK) / (1 + 0.1245 e^{-0.1 VF/RT} + 0.0353 e^{-VF/RT})
    double ncx_up, ncx_down;   // iNaCa = ncx_up Nai^3 - ncx_down Cai
    double ipk;          // gpK / (1 + exp((25 - V)/5.98))
};

__device__ __forceinline__ VOnly v_only(const cell::Coef &C, const IonicParams &P, double V)
{
    using namespace cell;
    VOnly o;
    // below -15 V e^{-phi} would leave the range; all that it enters has saturated
    const double phi = (V < -1.5e4 ? -1.5e4 : V) * (1.0 / RTONF);
    const double e1 = exp_(C, -phi), up = exp_(C, NCX_GAMMA * phi), down = up * e1;
    constexpr double nao3 = NA_O * NA_O * NA_O;
    constexpr double ncx_den = (KM_NAI * KM_NAI * KM_NAI + nao3) * (KM_CA + CA_O);
    // the pump's and the exchanger's denominators, and 1 + exp((25 - V)/5.98)
    const double rn = rcp(1.0 + 0.1245 * exp_(C, -0.1 * phi) + 0.0353 * e1);
    const double rx = rcp(ncx_den * (1.0 + K_SAT * down));
    o.nak = P.v[10] * (K_O / (K_O + KM_K)) * rn;
    o.ncx_up = P.v[11] * CA_O * (rx * up);
    o.ncx_down = P.v[11] * (nao3 * NCX_ALPHA) * (rx * down);
    const double w = (V - 15.0) * (2.0 / RTONF);
    double ew, em1;
    exp_expm1(C, clip(w, 700.0), ew, em1);
    o.ical_drive = w == 0.0 ? 2.0 * Far : 2.0 * Far * (w * rcp(em1));
    o.ical_ew = 0.25 * ew;
    o.ipk = P.v[9] * rcp(1.0 + exp_(C, (25.0 - clip(V, 2400.0)) * (1.0 / 5.98)));
    return o;
}

// Products of the gating variables that enter the currents, formed in FP64
// from the stored gates: the currents need these five numbers, not the
// twelve gates, which keeps the live set of a thread small.
struct GateProducts {
    double to;    // r s           (transient outward)
    double kr;    // xr1 xr2       (rapid delayed rectifier)
    double ks;    // xs^2          (slow delayed rectifier)
    double na;    // m^3 h j       (fast sodium)
    double cal;   // d f f2 fCass  (L-type calcium)
};

struct Currents {
    double iK1, ito, iKr, iKs, iCaL, iNaK, iNa, ibNa, iNaCa, ibCa, ipK, ipCa;
    __device__ double total() const
    {
        return iK1 + ito + iKr + iKs + iCaL + iNaK + iNa + ibNa + iNaCa + ibCa + ipK + ipCa;
    }
};

// currents at V and the concentration-type states c[0..5] (Ki Nai Cai CaSR
// CaSS Rbar) and gates summarised by gp
__device__ __forceinline__ Currents tt_currents(const cell::Coef &C, const IonicParams &P, double V,
                                                const VOnly &vo, const double *c,
                                                const GateProducts &gp)
{
    using namespace cell;
    const double gNa = P.v[0], gK1 = P.v[1], gto = P.v[2], gKr = P.v[3], gKs = P.v[4];
    const double gCaL = P.v[5], gbNa = P.v[6], gbCa = P.v[7], gpCa = P.v[8];
    const double ki = c[KI], nai = c[NAI], cai = c[CAI];
    const double e_k = RTONF * log_ratio(C, 1.6863989535702286, 7.914947588915769e-17, ki);
    const double e_na = RTONF * log_ratio(C, 4.941642422609304, 4.344622201918654e-16, nai);
    const double e_ks = RTONF * log_ratio(C, 2.2617630984737906, -9.075191670702233e-17, ki + P_KNA * nai);
    const double e_ca = 0.5 * RTONF * log_ratio(C, 0.6931471805599453, 2.3190468138462996e-17, cai);
    const double ko_scale = sqrt(K_O / 5.4);
    Currents cu;
    // inward rectifier: steady-state rectification a/(a+b) with
    // a = 0.1/(1+e1), b = q/(1+e2) and y = V - E_K: e1 = e^{0.06 y - 12},
    // e2 = e^{-0.5 y} = 1/T^5 with T = e^{0.1 y}; both denominators and T^5
    // cleared: 0.1 (1 + T^5) / (0.1 (1 + T^5) + T^5 q (1 + e1)).  Beyond
    // +-1000 mV the factor has saturated.
    const double y = clip(V - e_k, 1000.0);
    const double T = exp_(C, 0.1 * y), T2 = T * T, T5 = T2 * T2 * T;
    const double a_k1 = __builtin_fma(0.1, T5, 0.1);
    const double b_k1 = T5 * (3.0 * exp_(C, 0.0002 * (y + 100.0)) + 0.36787944117144233 * T)
                      * __builtin_fma(6.14421235332821e-06, exp_(C, 0.06 * y), 1.0);
    cu.iK1 = gK1 * ko_scale * (a_k1 * rcp(a_k1 + b_k1)) * (V - e_k);
    cu.ito = gto * gp.to * (V - e_k);
    cu.iKr = gKr * ko_scale * gp.kr * (V - e_k);
    cu.iKs = gKs * gp.ks * (V - e_ks);
    cu.iNa = gNa * gp.na * (V - e_na);
    cu.ibNa = gbNa * (V - e_na);
    cu.iCaL = gCaL * gp.cal * vo.ical_drive * (c[CASS] * vo.ical_ew - CA_O);
    cu.ibCa = gbCa * (V - e_ca);
    cu.iNaK = vo.nak * (nai * rcp(nai + KM_NA));
    cu.iNaCa = vo.ncx_up * (nai * nai * nai) - vo.ncx_down * cai;
    cu.ipCa = gpCa * (cai * rcp(K_PCA + cai));
    cu.ipK = vo.ipk * (V - e_k);
    return cu;
}

// Gating variables of the model advanced by Rush-Larsen at V^k in FP32,
// streamed one at a time: gate s (xr1 xr2 xs m h j d f f2 fCass s r) is
// read from g[s * ld], advanced and written back at once.  po and pn receive
// the gate products before and after the step; cass is CaSS^k.
__device__ __forceinline__ void tt_gates32(float V, float dt, float cass, float *__restrict__ g,
                                           int64_t ld, GateProducts &po, GateProducts &pn)
{
    using T = float;
    const T one = T(1);
    auto sqt = [](T x) { return x * x; };
    // advance gate s towards y_inf with time constant tau; old value to y0
    auto adv = [&](int s, T y_inf, T tau, double &y0) -> double {
        const T y = g[s * ld];
        const T y1 = rush_larsen(y, y_inf, tau, dt);
        g[s * ld] = y1;
        y0 = (double)y;
        return (double)y1;
    };
    auto adv_rate = [&](int s, T y_inf, T rate, double &y0) -> double {
        const T y = g[s * ld];
        const T y1 = rush_larsen_rate(y, y_inf, rate, dt);
        g[s * ld] = y1;
        y0 = (double)y;
        return (double)y1;
    };
    double o0, o1, o2, n0, n1, n2;

    // rapid delayed rectifier xr1, xr2
    {
        T inf = one / (one + expf((T(-26.0) - V) * T(1.0 / 7.0)));
        // 450/(1+a) * 6/(1+b) with one division
        T tau = T(450.0 * 6.0) / ((one + expf((T(-45.0) - V) * T(1.0 / 10.0))) * (one + expf((V + T(30.0)) * T(1.0 / 11.5))));
        n0 = adv(0, inf, tau, o0);
    }
    {
        T inf = one / (one + expf((V + T(88.0)) * T(1.0 / 24.0)));
        T tau = T(3.0 * 1.12) / ((one + expf((T(-60.0) - V) * T(1.0 / 20.0))) * (one + expf((V - T(60.0)) * T(1.0 / 20.0))));
        n1 = adv(1, inf, tau, o1);
    }
    po.kr = o0 * o1;
    pn.kr = n0 * n1;
    // slow delayed rectifier xs
    {
        T inf = one / (one + expf((T(-5.0) - V) * T(1.0 / 14.0)));
        T tau = T(1400.0) / (sqrtf(one + expf((T(5.0) - V) * T(1.0 / 6.0))) * (one + expf((V - T(35.0)) * T(1.0 / 15.0))))
              + T(80.0);
        n0 = adv(2, inf, tau, o0);
    }
    po.ks = o0 * o0;
    pn.ks = n0 * n0;
    // fast sodium m, h, j
    {
        T inf = one / sqt(one + expf((T(-56.86) - V) * T(1.0 / 9.03)));
        T tau = (one / (one + expf((T(-60.0) - V) * T(1.0 / 5.0))))
              * (T(0.1) / (one + expf((V + T(35.0)) * T(1.0 / 5.0))) + T(0.1) / (one + expf((V - T(50.0)) * T(1.0 / 200.0))));
        n0 = adv(3, inf, tau, o0);
    }
    {
        T h_inf = one / sqt(one + expf((V + T(71.55)) * T(1.0 / 7.43)));
        T alpha_h, beta_h, alpha_j, beta_j;
        if (V < T(-40.0)) {
            alpha_h = T(0.057) * expf(-(V + T(80.0)) * T(1.0 / 6.8));
            beta_h = T(2.7) * expf(T(0.079) * V) + T(3.1e5) * expf(T(0.3485) * V);
            alpha_j = (T(-25428.0) * expf(T(0.2444) * V) - T(6.948e-6) * expf(T(-0.04391) * V)) * (V + T(37.78))
                    / (one + expf(T(0.311) * (V + T(79.23))));
            beta_j = T(0.02424) * expf(T(-0.01052) * V) / (one + expf(T(-0.1378) * (V + T(40.14))));
        } else {
            alpha_h = T(0.0);
            beta_h = T(0.77 / 0.13) / (one + expf(-(V + T(10.66)) * T(1.0 / 11.1)));
            alpha_j = T(0.0);
            beta_j = T(0.6) * expf(T(0.057) * V) / (one + expf(T(-0.1) * (V + T(32.0))));
        }
        n1 = adv_rate(4, h_inf, alpha_h + beta_h, o1);
        n2 = adv_rate(5, h_inf, alpha_j + beta_j, o2);
    }
    po.na = o0 * o0 * o0 * o1 * o2;
    pn.na = n0 * n0 * n0 * n1 * n2;
    // L-type calcium d, f, f2, fCass
    {
        T inf = one / (one + expf((T(-8.0) - V) * T(1.0 / 7.5)));
        T tau = (T(1.4) / (one + expf((T(-35.0) - V) * T(1.0 / 13.0))) + T(0.25)) * (T(1.4) / (one + expf((V + T(5.0)) * T(1.0 / 5.0))))
              + one / (one + expf((T(50.0) - V) * T(1.0 / 20.0)));
        n0 = adv(6, inf, tau, o0);
    }
    {
        T inf = one / (one + expf((V + T(20.0)) * T(1.0 / 7.0)));
        T tau = T(1102.5) * expf(-sqt(V + T(27.0)) * T(1.0 / 225.0)) + T(200.0) / (one + expf((T(13.0) - V) * T(1.0 / 10.0)))
              + T(180.0) / (one + expf((V + T(30.0)) * T(1.0 / 10.0))) + T(20.0);
        n1 = adv(7, inf, tau, o1);
    }
    po.cal = o0 * o1;
    pn.cal = n0 * n1;
    {
        T inf = T(0.67) / (one + expf((V + T(35.0)) * T(1.0 / 7.0))) + T(0.33);
        T tau = T(562.0) * expf(-sqt(V + T(27.0)) * T(1.0 / 240.0)) + T(31.0) / (one + expf((T(25.0) - V) * T(1.0 / 10.0)))
              + T(80.0) / (one + expf((V + T(30.0)) * T(1.0 / 10.0)));
        n0 = adv(8, inf, tau, o0);
    }
    {
        T ratio2 = sqt(cass * T(1.0 / 0.05));
        T inf = T(0.6) / (one + ratio2) + T(0.4);
        T tau = T(80.0) / (one + ratio2) + T(2.0);
        n1 = adv(9, inf, tau, o1);
    }
    po.cal = po.cal * o0 * o1;
    pn.cal = pn.cal * n0 * n1;
    // transient outward s (endocardial), r
    {
        T inf = one / (one + expf((V + T(28.0)) * T(1.0 / 5.0)));
        T tau = T(1000.0) * expf(-sqt(V + T(67.0)) * T(1.0 / 1000.0)) + T(8.0);
        n0 = adv(10, inf, tau, o0);
    }
    {
        T inf = one / (one + expf((T(20.0) - V) * T(1.0 / 6.0)));
        T tau = T(9.5) * expf(-sqt(V + T(40.0)) * T(1.0 / 1800.0)) + T(0.8);
        n1 = adv(11, inf, tau, o1);
    }
    po.to = o1 * o0;
    pn.to = n1 * n0;
}

// The same gates in FP64 with fewer operations: the sigmoids' exponentials
// share a few bases (e^{V/20} gives those of V/10, e^{V/14} those of V/7,
// e^{V/15} those of V/7.5, reciprocals their inverses) and every time constant
// enters as its rate with the denominators cleared.  V is held within
// +-2400 mV, beyond which every gate has saturated, so that no product of two
// denominators overflows.  The m gate keeps exponentials of its own: its
// steep time constant makes the current feel the rounding of e^{V/5}'s larger
// argument.
__device__ __forceinline__ void tt_gates64(const cell::Coef &C, double V, double dt, double cass,
                                           double *__restrict__ g, int64_t ld, GateProducts &po,
                                           GateProducts &pn)
{
    using namespace cell;
    const double ndt = -dt;
    // gates are loaded three ahead of their use
    double gy[12];
#pragma unroll
    for (int k = 0; k < 3; ++k) gy[k] = g[k * ld];
    // advance gate s towards inf at the rate 1/tau; old value to y0
    auto adv = [&](int s, double inf, double rate, double &y0) -> double {
        y0 = gy[s];
        if (s + 3 < 12) gy[s + 3] = g[(s + 3) * ld];
        const double y1 = inf - (inf - y0) * exp_neg(C, ndt * rate);
        g[s * ld] = y1;
        return y1;
    };
    const double v = clip(V, 2400.0);
    const double E20 = exp_(C, v * (1.0 / 20.0)), E14 = exp_(C, v * (1.0 / 14.0));
    const double E15 = exp_(C, v * (1.0 / 15.0));
    const double I20 = rcp(E20), I14 = rcp(E14), I15 = rcp(E15);
    const double E10 = E20 * E20, I10 = I20 * I20;
    const double E5 = exp_(C, v * (1.0 / 5.0));
    const double E7 = E14 * E14, I7 = I14 * I14;
    const double I6 = exp_(C, v * (-1.0 / 6.0));
    auto one = [](double c, double E) { return __builtin_fma(c, E, 1.0); };   // 1 + c E
    double o0, o1, o2, n0, n1, n2, ra, rb;

    // rapid delayed rectifier xr1, xr2
    ra = rcp(one(0.0243728440732796, I7));
    rb = rcp(1.0 + exp_(C, (v + 88.0) * (1.0 / 24.0)));
    n0 = adv(0, ra, one(0.011108996538242306, I10) * (1.0 + exp_(C, (v + 30.0) * (1.0 / 11.5)))
                        * (1.0 / 2700.0), o0);
    n1 = adv(1, rb, one(0.049787068367863944, I20) * one(0.049787068367863944, E20)
                        * (1.0 / (3.0 * 1.12)), o1);
    po.kr = o0 * o1;
    pn.kr = n0 * n1;
    // slow delayed rectifier xs
    {
        const double f = sqrt(one(2.300975890892825, I6)) * one(0.09697196786440507, E15);
        ra = rcp(one(0.6996725373751304, I14));
        rb = rcp(__builtin_fma(80.0, f, 1400.0));
        n0 = adv(2, ra, f * rb, o0);
    }
    po.ks = o0 * o0;
    pn.ks = n0 * n0;
    // fast sodium m, h, j
    {
        // (1/5 with what its rounding leaves: that times the exponents' size is a
        // third of m's rms error, 3.4e-16 without at dt 0.005, 2.5e-16 with it,
        // 3.1e-16 with library functions and divisions throughout)
        const double q = 1.0 + exp_(C, (-56.86 - v) * (1.0 / 9.03));
        const double e1 = exp_(C, times(-60.0 - v, 0.2, -0x1.999999999999ap-57));
        const double e2 = exp_(C, times(v + 35.0, 0.2, -0x1.999999999999ap-57)), e3 = exp_(C, (v - 50.0) * (1.0 / 200.0));
        ra = rcp(q * q);
        rb = rcp(2.0 + e2 + e3);
        n0 = adv(3, ra, 10.0 * (1.0 + e1) * (1.0 + e2) * (1.0 + e3) * rb, o0);
    }
    {
        const double q = 1.0 + exp_(C, (v + 71.55) * (1.0 / 7.43)), q2 = q * q;
        double rate_h, rate_j;
        if (v < -40.0) {
            const double da = 1.0 + exp_(C, 0.311 * (v + 79.23)), db = 1.0 + exp_(C, -0.1378 * (v + 40.14));
            rate_h = 0.057 * exp_(C, (v + 80.0) * (-1.0 / 6.8))
                   + (2.7 * exp_(C, 0.079 * v) + 3.1e5 * exp_(C, 0.3485 * v));
            rate_j = (-25428.0 * exp_(C, 0.2444 * v) - 6.948e-6 * exp_(C, -0.04391 * v)) * (v + 37.78)
                         * rcp(da)
                   + 0.02424 * exp_(C, -0.01052 * v) * rcp(db);
        } else {
            const double dh = 1.0 + exp_(C, (v + 10.66) * (-1.0 / 11.1)), dj = one(0.04076220397836622, I10);
            rate_h = (0.77 / 0.13) * rcp(dh);
            rate_j = 0.6 * exp_(C, 0.057 * v) * rcp(dj);
        }
        n1 = adv(4, rcp(q2), rate_h, o1);
        n2 = adv(5, rcp(q2), rate_j, o2);
    }
    po.na = o0 * o0 * o0 * o1 * o2;
    pn.na = n0 * n0 * n0 * n1 * n2;
    // L-type calcium d, f, f2, fCass
    {
        const double p = 1.0 + exp_(C, (-35.0 - v) * (1.0 / 13.0)), q = one(2.718281828459045, E5);
        const double t = one(12.182493960703473, I20), pq = p * q;
        ra = rcp(one(0.34415378686541237, I15 * I15));
        rb = rcp(1.4 * __builtin_fma(0.25, p, 1.4) * t + pq);
        n0 = adv(6, ra, pq * t * rb, o0);
    }
    const double b = one(20.085536923187668, E10), x27 = sq(v + 27.0);
    {
        const double a = one(3.669296667619244, I10), ab = a * b;
        const double den = __builtin_fma(1102.5, exp_(C, x27 * (-1.0 / 225.0)), 20.0) * ab
                         + (200.0 * b + 180.0 * a);
        ra = rcp(one(17.41170806332765, E7));
        rb = rcp(den);
        n1 = adv(7, ra, ab * rb, o1);
    }
    po.cal = o0 * o1;
    pn.cal = n0 * n1;
    {
        const double a = one(12.182493960703473, I10), ab = a * b;
        const double den = 562.0 * exp_(C, x27 * (-1.0 / 240.0)) * ab + (31.0 * b + 80.0 * a);
        ra = rcp(one(148.4131591025766, E7));
        rb = rcp(den);
        n0 = adv(8, __builtin_fma(0.67, ra, 0.33), ab * rb, o0);
    }
    {
        const double f = 1.0 + sq(cass * (1.0 / 0.05));
        ra = rcp(f);
        rb = rcp(__builtin_fma(2.0, f, 80.0));
        n1 = adv(9, __builtin_fma(0.6, ra, 0.4), f * rb, o1);
    }
    po.cal = po.cal * o0 * o1;
    pn.cal = pn.cal * n0 * n1;
    // transient outward s (endocardial), r
    ra = rcp(one(270.42640742615265, E5));
    rb = rcp(__builtin_fma(1000.0, exp_(C, sq(v + 67.0) * (-1.0 / 1000.0)), 8.0));
    n0 = adv(10, ra, rb, o0);
    ra = rcp(one(28.031624894526136, I6));
    rb = rcp(__builtin_fma(9.5, exp_(C, sq(v + 40.0) * (-1.0 / 1800.0)), 0.8));
    n1 = adv(11, ra, rb, o1);
    po.to = o1 * o0;
    pn.to = n1 * n0;
}

// One step of the model at one node: concentration-type states c[0..5]
// (Ki Nai Cai CaSR CaSS Rbar) by forward Euler in FP64, gates (g[s * ld],
// s = 0..11) by Rush-Larsen in precision G; returns I_ion(V^k, u^{k+1}) / Cm
// in FP64.
template <typename G>
__device__ double tt_point(const IonicParams &P, double dt, double V, double *c,
                           G *__restrict__ g, int64_t ld)
{
    const cell::Coef C = cell::make_coef();
    const double cai = c[CAI], casr = c[CASR], cass = c[CASS], rbar = c[RBAR];

    // ---- gating variables at V^k (their products at u^k and u^{k+1}) ----
    GateProducts po, pn;
    if constexpr (sizeof(G) == sizeof(double))
        tt_gates64(C, V, dt, cass, g, ld, po, pn);
    else
        tt_gates32((float)V, (float)dt, (float)cass, g, ld, po, pn);
    const VOnly vo = v_only(C, P, V);

    // ---- calcium subsystem and ion concentrations: rates at (V^k, u^k) ----
    // (quotients with their denominators cleared)
    const Currents cur = tt_currents(C, P, V, vo, c, po);
    const double casr2 = casr * casr, cai2 = cai * cai;
    const double xc = sq(cai + KBUF_C), xsr = sq(casr + KBUF_SR), xss = sq(cass + KBUF_SS);
    const double r_sr = cell::rcp(casr2 + EC_SR * EC_SR);
    const double r_up = cell::rcp(cai2 + K_UP * K_UP);
    const double r_c = cell::rcp(xc + BUF_C * KBUF_C);
    const double r_bsr = cell::rcp(xsr + BUF_SR * KBUF_SR);
    const double kcasr = MAX_SR - (MAX_SR - MIN_SR) * (casr2 * r_sr);
    const double k1c2 = K1_PRIME * cass * cass;
    const double r_ss = cell::rcp(xss + BUF_SS * KBUF_SS);
    const double r_open = cell::rcp(K3 * kcasr + k1c2);
    double i_rel = V_REL * (k1c2 * rbar * r_open) * (casr - cass);
    double i_up = VMAX_UP * (cai2 * r_up);
    double i_leak = V_LEAK * (casr - cai);
    double i_xfer = V_XFER * (cass - cai);
    double d_rbar = -(K2_PRIME * kcasr) * cass * rbar + K4 * (1.0 - rbar);
    double d_cai = (xc * r_c) * ((i_leak - i_up) * (VOLSR / VOLC) + i_xfer
                            - (cur.ibCa + cur.ipCa - 2.0 * cur.iNaCa) * (CAPAC / (2.0 * VOLC * Far)));
    double d_casr = (xsr * r_bsr) * (i_up - i_rel - i_leak);
    double d_cass = (xss * r_ss) * (-cur.iCaL * (CAPAC / (2.0 * VOLSS * Far)) + i_rel * (VOLSR / VOLSS)
                              - i_xfer * (VOLC / VOLSS));
    double d_nai = -(cur.iNa + cur.ibNa + 3.0 * cur.iNaK + 3.0 * cur.iNaCa) * (CAPAC / (VOLC * Far));
    double d_ki = -(cur.iK1 + cur.ito + cur.iKr + cur.iKs - 2.0 * cur.iNaK + cur.ipK) * (CAPAC / (VOLC * Far));

    // ---- forward Euler for the concentration-type states ----
    c[KI] = c[KI] + dt * d_ki;
    c[NAI] = c[NAI] + dt * d_nai;
    c[CAI] = cai + dt * d_cai;
    c[CASR] = casr + dt * d_casr;
    c[CASS] = cass + dt * d_cass;
    c[RBAR] = rbar + dt * d_rbar;

    // ---- I_ion(V^k, u^{k+1}) ----
    return tt_currents(C, P, V, vo, c, pn).total();
}

// ---------------------------------------------------------------------------
// Courtemanche-Ramirez-Nattel 1998 human atrial cell (Am. J. Physiol. 275:
// H301), 20 states + V:
//   Na_i K_i Ca_i Ca_up Ca_rel (mM; forward Euler)
//   m h j oa oi ua ui xr xs d f fCa u v w (Rush-Larsen)
// params: gNa gK1 gto gKr gKs gCaL gbNa gbCa (nS/pF), INaK_max INaCa_max
// IpCa_max (pA/pF), Iup_max (mM/ms), and a scale of gKur(V).
// Currents are per unit capacitance; the membrane capacitance (100 pF) turns
// them into the pA that the concentration balances and the release trigger
// use.
// ---------------------------------------------------------------------------
namespace crn {
constexpr double RT_F = 8.3143 * 310.0 / 96.4867;   // mV
constexpr double FARADAY = 96.4867;                   // C/mmol
constexpr double CAP = 100.0;                         // pF
constexpr double VOL_I = 13668.0, VOL_UP = 1109.52, VOL_REL = 96.48;   // um^3
constexpr double K_OUT = 5.4, NA_OUT = 140.0, CA_OUT = 1.8;
constexpr double NAK_KM_NA_3_2 = 31.622776601683793, NAK_KM_K = 1.5;   // 10 mM to the 3/2
constexpr double NACA_KM_NA = 87.5, NACA_KM_CA = 1.38, NACA_SAT = 0.1, NACA_GAMMA = 0.35;
constexpr double REL_RATE = 30.0, UP_KM = 0.00092, UP_CA_MAX = 15.0, TR_TAU = 180.0;
constexpr double CMDN_TOT = 0.05, CMDN_KM = 0.00238, TRPN_TOT = 0.07, TRPN_KM = 0.0005;
constexpr double CSQN_TOT = 10.0, CSQN_KM = 0.8;
constexpr double Q10 = 3.0;
constexpr double V_REST = -81.18;
// ratio of the sodium-potassium pump's [Na]_o dependence, (e^{Na_o/67.3} - 1) / 7
__device__ __forceinline__ double nak_sigma() { return (exp(NA_OUT / 67.3) - 1.0) / 7.0; }
}  // namespace crn
constexpr int CRN_NS = 20;
constexpr int CRN_NP = 13;
__device__ const double CRN_U0[CRN_NS] = {11.17,  139.0,  1.013e-4, 1.488,    1.488,
                                          2.908e-3, 0.9649, 0.9775, 3.043e-2, 0.9992,
                                          4.966e-3, 0.9986, 3.296e-5, 1.869e-2, 1.367e-4,
                                          0.9996, 0.7755, 0.0,      1.0,      0.9992};

// x / (1 - e^{-x/s}), whose limit at x = 0 is s; e receives e^{-x/s}.  xe stands
// in for x in the exponential: x held in its range
__device__ __forceinline__ double rise_ratio(const cell::Coef &C, double x, double xe, double s, double &e)
{
    double em1;
    cell::exp_expm1(C, -xe * (1.0 / s), e, em1);
    return x != 0.0 ? cell::div(x, -em1) : s;
}
// x / (e^{x/s} - 1), whose limit at x = 0 is s
__device__ __forceinline__ double fall_ratio(const cell::Coef &C, double x, double xe, double s)
{
    double e, em1;
    cell::exp_expm1(C, xe * (1.0 / s), e, em1);
    return x != 0.0 ? cell::div(x, em1) : s;
}
// 1 / (1 + e^{-x}), |x| < 700
__device__ __forceinline__ double logistic(const cell::Coef &C, double x)
{
    return cell::rcp(1.0 + cell::exp_(C, -x));
}

struct CrnCurrents {
    double iNa, iK1, ito, iKur, iKr, iKs, iCaL, iNaK, iNaCa, ibNa, ibCa, ipCa;
    __device__ double total() const
    {
        return ((iNa + ibNa) + (iK1 + ito + iKur + iKr + iKs)) + ((iCaL + ibCa + ipCa) + (iNaK + iNaCa));
    }
};

// products of the gates that enter the currents
struct CrnGates {
    double na;    // m^3 h j
    double to;    // oa^3 oi
    double kur;   // ua^3 ui
    double kr;    // xr
    double ks;    // xs
    double cal;   // d f fCa
};

// currents at V, concentrations y[0..2] and gates summarised by gp
__device__ __forceinline__ CrnCurrents crn_currents(const cell::Coef &C, const IonicParams &P, double V,
                                                    const double *y, const CrnGates &gp)
{
    using namespace crn;
    using namespace cell;
    const double na = y[0], k = y[1], ca = y[2];
    const double e_na = RT_F * log_ratio(C, 4.941642422609304, 4.344622201918654e-16, na), e_k = RT_F * log_ratio(C, 1.6863989535702286, 7.914947588915769e-17, k);
    const double e_ca = 0.5 * RT_F * log_ratio(C, 0.5877866649021191, -5.2182156685858313e-17, ca);
    const double v = clip(V, 9e3), u = v * (1.0 / RT_F);   // every exponential but e_in stays in range
    CrnCurrents c;
    c.iNa = P.v[0] * gp.na * (V - e_na);
    c.iK1 = P.v[1] * (V - e_k) * logistic(C, -0.07 * (v + 80.0));
    c.ito = P.v[2] * gp.to * (V - e_k);
    const double g_kur = P.v[12] * (0.005 + 0.05 * logistic(C, (v - 15.0) * (1.0 / 13.0)));
    c.iKur = g_kur * gp.kur * (V - e_k);
    c.iKr = P.v[3] * gp.kr * (V - e_k) * logistic(C, (v + 15.0) * (-1.0 / 22.4));
    c.iKs = P.v[4] * (gp.ks * gp.ks) * (V - e_k);
    c.iCaL = P.v[5] * gp.cal * (V - 65.0);
    const double pump_v = rcp(1.0 + 0.1245 * exp_(C, -0.1 * u) + 0.0365 * nak_sigma() * exp_(C, -u));
    // 1 / (1 + (K_m / Na)^{3/2}), defined without sodium too
    const double na_3_2 = na * sqrt(na);
    const double pump_na = na_3_2 * rcp(na_3_2 + NAK_KM_NA_3_2);
    c.iNaK = P.v[8] * pump_v * pump_na * (K_OUT / (K_OUT + NAK_KM_K));
    const double e_in = exp_(C, NACA_GAMMA * (V * (1.0 / RT_F))), e_out = exp_(C, (NACA_GAMMA - 1.0) * u);
    const double km3 = NACA_KM_NA * NACA_KM_NA * NACA_KM_NA, nao3 = NA_OUT * NA_OUT * NA_OUT;
    c.iNaCa = div(P.v[9] * (e_in * (na * na * na) * CA_OUT - e_out * nao3 * ca),
                  (km3 + nao3) * (NACA_KM_CA + CA_OUT) * (1.0 + NACA_SAT * e_out));
    c.ibNa = P.v[6] * (V - e_na);
    c.ibCa = P.v[7] * (V - e_ca);
    c.ipCa = P.v[10] * (ca * rcp(0.0005 + ca));
    return c;
}

// One step at one node: concentrations y[0..4] (Na_i K_i Ca_i Ca_up Ca_rel)
// by forward Euler, gates g[s * ld] (m h j oa oi ua ui xr xs d f fCa u v w) by
// Rush-Larsen, streamed one at a time: the currents need six products of them.
// Fluxes and rates at (V^k, u^k); returns I_ion(V^k, u^{k+1}) / Cm (mV/ms).
__device__ double crn_point(const IonicParams &P, double dt, double V, double *y,
                            double *__restrict__ g, int64_t ld)
{
    using namespace crn;
    using namespace cell;
    const Coef C = make_coef();
    // ---- gates: Rush-Larsen with the rate 1/tau at V^k, which is held within
    // +-3000 mV in the exponentials: none overflows, and every gate's limit and
    // what they give of its rate have saturated there ----
    const double v = clip(V, 3000.0), ndt = -dt;
    // gates are loaded three ahead of their use
    double gy[15];
#pragma unroll
    for (int k = 0; k < 3; ++k) gy[k] = g[k * ld];
    // advance gate s towards inf at the given rate; old value to y0
    auto adv = [&](int s, double inf, double rate, double &y0) -> double {
        y0 = gy[s];
        if (s + 3 < 15) gy[s + 3] = g[(s + 3) * ld];
        const double y1 = inf - (inf - y0) * exp_neg(C, ndt * rate);
        g[s * ld] = y1;
        return y1;
    };
    CrnGates po, pn;
    double e, o0, o1, o2, n0, n1, n2;
    {   // fast sodium m, h, j from their opening and closing rates
        const double am = 0.32 * rise_ratio(C, V + 47.13, v + 47.13, 10.0, e), bm = 0.08 * exp_(C, v * (-1.0 / 11.0));
        n0 = adv(0, div(am, am + bm), am + bm, o0);
        double ah = 0.0, bh, aj = 0.0, bj;
        if (v < -40.0) {
            ah = 0.135 * exp_(C, (v + 80.0) * (-1.0 / 6.8));
            bh = 3.56 * exp_(C, 0.079 * v) + 3.1e5 * exp_(C, 0.35 * v);
            aj = (-127140.0 * exp_(C, 0.2444 * v) - 3.474e-5 * exp_(C, -0.04391 * v)) * (v + 37.78)
               * logistic(C, -0.311 * (v + 79.23));
            bj = 0.1212 * exp_(C, -0.01052 * v) * logistic(C, 0.1378 * (v + 40.14));
        } else {
            bh = (1.0 / 0.13) * logistic(C, (v + 10.66) * (1.0 / 11.1));
            bj = 0.3 * exp_(C, -2.535e-7 * V) * logistic(C, 0.1 * (v + 32.0));
        }
        n1 = adv(1, div(ah, ah + bh), ah + bh, o1);
        n2 = adv(2, div(aj, aj + bj), aj + bj, o2);
        po.na = o0 * o0 * o0 * o1 * o2;
        pn.na = n0 * n0 * n0 * n1 * n2;
    }
    {   // transient (oa, oi) and ultrarapid (ua, ui) potassium, Q10 = 3
        const double a_a = 0.65 * rcp(exp_(C, (v + 10.0) * (-1.0 / 8.5)) + exp_(C, (v - 30.0) * (-1.0 / 59.0)));
        const double b_a = 0.65 * rcp(2.5 + exp_(C, (v + 82.0) * (1.0 / 17.0)));
        const double r_a = (a_a + b_a) * Q10;
        n0 = adv(3, logistic(C, (v + 20.47) * (1.0 / 17.54)), r_a, o0);
        const double a_oi = rcp(18.53 + exp_(C, (v + 113.7) * (1.0 / 10.95)));
        const double b_oi = rcp(35.56 + exp_(C, (v + 1.26) * (-1.0 / 7.44)));
        n1 = adv(4, logistic(C, (v + 43.1) * (-1.0 / 5.3)), (a_oi + b_oi) * Q10, o1);
        po.to = o0 * o0 * o0 * o1;
        pn.to = n0 * n0 * n0 * n1;
        n0 = adv(5, logistic(C, (v + 30.3) * (1.0 / 9.6)), r_a, o0);
        const double a_ui = rcp(21.0 + exp_(C, (v - 185.0) * (-1.0 / 28.0)));
        const double b_ui = exp_(C, (v - 158.0) * (1.0 / 16.0));
        n1 = adv(6, logistic(C, (v - 99.45) * (-1.0 / 27.48)), (a_ui + b_ui) * Q10, o1);
        po.kur = o0 * o0 * o0 * o1;
        pn.kur = n0 * n0 * n0 * n1;
    }
    {   // rapid and slow delayed rectifiers
        const double a_r = 0.0003 * rise_ratio(C, V + 14.1, v + 14.1, 5.0, e);
        const double b_r = 7.3898e-5 * fall_ratio(C, V - 3.3328, v - 3.3328, 5.1237);
        pn.kr = adv(7, logistic(C, (v + 14.1) * (1.0 / 6.5)), a_r + b_r, po.kr);
        const double a_s = 4e-5 * rise_ratio(C, V - 19.9, v - 19.9, 17.0, e);
        const double b_s = 3.5e-5 * fall_ratio(C, V - 19.9, v - 19.9, 9.0);
        pn.ks = adv(8, sqrt(logistic(C, (v - 19.9) * (1.0 / 12.7))), 2.0 * (a_s + b_s), po.ks);
    }
    {   // L-type calcium d, f, fCa
        const double x = v + 10.0;
        // 1/tau_d = 0.035 x (1 + e^{-x/6.24}) / (1 - e^{-x/6.24})
        const double r_x = rise_ratio(C, V + 10.0, x, 6.24, e), r_d = 0.035 * r_x * (1.0 + e);
        n0 = adv(9, logistic(C, x * (1.0 / 8.0)), r_d, o0);
        const double r_f = (0.0197 * exp_(C, -(0.0337 * 0.0337) * x * x) + 0.02) * (1.0 / 9.0);
        n1 = adv(10, logistic(C, (v + 28.0) * (-1.0 / 6.9)), r_f, o1);
        n2 = adv(11, rcp(1.0 + y[2] * (1.0 / 0.00035)), 0.5, o2);
        po.cal = o0 * o1 * o2;
        pn.cal = n0 * n1 * n2;
    }

    // ---- currents and fluxes at (V^k, u^k) ----
    const CrnCurrents c = crn_currents(C, P, V, y, po);
    const double ca = y[2], ca_up = y[3], ca_rel = y[4];
    const double uu = gy[12];
    const double j_rel = REL_RATE * (uu * uu) * gy[13] * gy[14] * (ca_rel - ca);
    const double j_tr = (ca_up - ca_rel) * (1.0 / TR_TAU);
    const double j_up = P.v[11] * (ca * rcp(ca + UP_KM));
    const double j_leak = P.v[11] * ca_up * (1.0 / UP_CA_MAX);
    // current (pA/pF) to concentration rate in the myoplasm (mM/ms)
    constexpr double to_conc = CAP / (FARADAY * VOL_I);
    const double d_na = -to_conc * (3.0 * (c.iNaK + c.iNaCa) + c.ibNa + c.iNa);
    const double d_k = to_conc * (2.0 * c.iNaK - (c.iK1 + c.ito + c.iKur + c.iKr + c.iKs));
    const double free_ca = 0.5 * to_conc * (2.0 * c.iNaCa - c.ipCa - c.iCaL - c.ibCa)
                         + (VOL_UP * (j_leak - j_up) + VOL_REL * j_rel) * (1.0 / VOL_I);
    // free_ca / (1 + buffering by troponin and calmodulin), denominators cleared
    const double x_cmdn = sq(ca + CMDN_KM), x_trpn = sq(ca + TRPN_KM), x_both = x_cmdn * x_trpn;
    const double d_ca = free_ca * x_both
                      * rcp(x_both + (TRPN_TOT * TRPN_KM) * x_cmdn + (CMDN_TOT * CMDN_KM) * x_trpn);
    const double d_up = j_up - j_leak - j_tr * (VOL_REL / VOL_UP);
    const double x_csqn = sq(ca_rel + CSQN_KM);
    const double d_rel = (j_tr - j_rel) * x_csqn * rcp(x_csqn + CSQN_TOT * CSQN_KM);

    // release trigger: SR release plus the Ca entry of I_CaL and I_NaCa (pA)
    const double fn = 1e-12 * VOL_REL * j_rel - (5e-13 / FARADAY) * CAP * (0.5 * c.iCaL - 0.2 * c.iNaCa);
    const double on_u = logistic(C, clip((fn - 3.4175e-13) * (1.0 / 13.67e-16), 700.0));

    {   // SR release gates u, v (trigger fn) and w (voltage)
        adv(12, on_u, 1.0 / 8.0, o0);
        const double v_inf = 1.0 - logistic(C, clip((fn - 6.835e-14) * (1.0 / 13.67e-16), 700.0));
        adv(13, v_inf, rcp(1.91 + 2.09 * on_u), o0);
        // 1/tau_w = x (1 + 0.3 e^{-x/5}) / (6 (1 - e^{-x/5}))
        const double r_x = rise_ratio(C, V - 7.9, v - 7.9, 5.0, e), r_w = r_x * (1.0 + 0.3 * e) * (1.0 / 6.0);
        adv(14, 1.0 - logistic(C, (v - 40.0) * (1.0 / 17.0)), r_w, o0);
    }
    // ---- forward Euler for the concentrations ----
    y[0] += dt * d_na;
    y[1] += dt * d_k;
    y[2] = ca + dt * d_ca;
    y[3] = ca_up + dt * d_up;
    y[4] = ca_rel + dt * d_rel;
    return crn_currents(C, P, V, y, pn).total();
}

// Row i holds a cell: i < n, or, with the per-tile count of real rows of the
// batched layout (padding rows at the end of each instance's last tile),
// (i mod TILE) < tile_real[i / TILE].
__device__ __forceinline__ bool real_row(int64_t i, int64_t n, const int32_t *tile_real)
{
    return tile_real ? (int)(i & (TILE - 1)) < tile_real[i / TILE] : i < n;
}

// The right-hand side's gathered values of row i, written where they are
// formed: as a kernel of its own this pass read V, V_prev and the source again
// (12 us of a step of 1,310,736 nodes, 4 of 232,472).
__device__ __forceinline__ void put_gather(const GatherOut &g, int64_t i, double v, double src,
                                           double vprev)
{
    g.gv[3 * i] = g.cm * v + g.dt * src;
    g.gv[3 * i + 1] = v;
    g.gv[3 * i + 2] = g.warm_start == 1 ? 2.0 * v - vprev : v;
}

// ---------------------------------------------------------------------------
// The ten Tusscher-Panfilov and Courtemanche-Ramirez-Nattel updates were bound
// by instruction issue: ~4,000 vector instructions a wavefront, half of them
// the library's exponentials, logarithms and divisions.  With the functions of
// cell:: and shared exponentials it is ~1,700, and the state traffic (18 or 20
// rows read and written) bounds the large sizes: at 1,255,450 cells 180 -> 117
// us and 178 -> 123 us (392 and 432 MB: 82 and 90 us at the copy rate), at
// 300,007 58 -> 41 and 55 -> 42 us.  Gates are streamed, loaded three ahead of
// their use: 106 and 118 registers, four wavefronts per SIMD with no spills
// (with the CRN states held in registers it was 179 and two wavefronts, 134 us).
template <int KIND, bool GATHER>
__global__ __launch_bounds__(256) void k_ionic_step(IonicParams P, int64_t n, int64_t ld, double dt,
                                                    double cm, const double *__restrict__ V,
                                                    double *__restrict__ u,
                                                    const double *__restrict__ istim,
                                                    double *__restrict__ out, int raw,
                                                    const int32_t *__restrict__ tile_real,
                                                    const int32_t *__restrict__ guard,
                                                    StepTimes times, GatherOut gather)
{
    if (guard && !*guard) return;   // enqueued ahead of a solve that is not done
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (!real_row(i, n, tile_real)) {
        if constexpr (GATHER)
            put_gather(gather, i, 0.0, 0.0, 0.0);
        else
            out[i] = 0.0;
        return;
    }
    double v = V[i];
    if (times.lat && !update_times(i, times.t1, times.Vold[i], v, times.lat, times.lrt))
        times.sc->nonfinite_v = 1;
    double iion = 0.0;
    if constexpr (KIND == MDX_KIND_MS) {
        double h = u[i];
        iion = ms_point<double>(P, dt, v, h);
        u[i] = h;
    } else if constexpr (KIND == MDX_KIND_TT) {
        double c[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) c[s] = u[s * ld + i];
        iion = tt_point<double>(P, dt, v, c, u + 6 * ld + i, ld);
#pragma unroll
        for (int s = 0; s < 6; ++s) u[s * ld + i] = c[s];
    } else if constexpr (KIND == MDX_KIND_CRN) {
        double c[5];
#pragma unroll
        for (int s = 0; s < 5; ++s) c[s] = u[s * ld + i];
        iion = crn_point(P, dt, v, c, u + 5 * ld + i, ld);
#pragma unroll
        for (int s = 0; s < 5; ++s) u[s * ld + i] = c[s];
    }
    if (raw) {
        out[i] = iion;
        return;
    }
    const double src = (istim ? istim[i] : 0.0) - cm * iion;
    if constexpr (GATHER)
        put_gather(gather, i, v, src, gather.Vprev[i]);
    else
        out[i] = src;
}

template <int KIND>
__global__ __launch_bounds__(256) void k_ionic_init(IonicParams P, int64_t n, int64_t ld,
                                                    double *__restrict__ V,
                                                    double *__restrict__ Vprev,
                                                    double *__restrict__ u,
                                                    const int32_t *__restrict__ tile_real)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ld) return;
    const bool real = real_row(i, n, tile_real);
    double v0 = 0.0;
    if constexpr (KIND == MDX_KIND_MS) {
        v0 = P.v[5];
        if (u) u[i] = real ? 1.0 : 0.0;
    } else if constexpr (KIND == MDX_KIND_TT) {
        v0 = TT_V_REST;
        if (u)
            for (int s = 0; s < TT_NS; ++s) u[s * ld + i] = real ? TT_U0[s] : 0.0;
    } else if constexpr (KIND == MDX_KIND_CRN) {
        v0 = crn::V_REST;
        // padding rows hold the rest state too (finite logarithms if read)
        if (u)
            for (int s = 0; s < CRN_NS; ++s) u[s * ld + i] = CRN_U0[s];
    }
    V[i] = real ? v0 : 0.0;
    Vprev[i] = real ? v0 : 0.0;
}

// Mixed-precision form: gating variables stored and advanced in FP32
// (g32[s * ld + i], s over the model's gates), concentration-type states and
// the current in FP64 (u[s * ld + i], rows 0..5 for the ten Tusscher-Panfilov
// model; Mitchell-Schaeffer has only its gate h).
template <int KIND, bool GATHER>
__global__ __launch_bounds__(256) void k_ionic_step_mixed(IonicParams P, int64_t n, int64_t ld,
                                                          double dt, double cm,
                                                          const double *__restrict__ V,
                                                          double *__restrict__ u,
                                                          float *__restrict__ g32,
                                                          const double *__restrict__ istim,
                                                          double *__restrict__ out,
                                                          const int32_t *__restrict__ tile_real,
                                                          const int32_t *__restrict__ guard,
                                                          StepTimes times, GatherOut gather)
{
    if (guard && !*guard) return;   // enqueued ahead of a solve that is not done
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (!real_row(i, n, tile_real)) {
        if constexpr (GATHER)
            put_gather(gather, i, 0.0, 0.0, 0.0);
        else
            out[i] = 0.0;
        return;
    }
    const double v = V[i];
    if (times.lat && !update_times(i, times.t1, times.Vold[i], v, times.lat, times.lrt))
        times.sc->nonfinite_v = 1;
    double iion = 0.0;
    if constexpr (KIND == MDX_KIND_MS) {
        float h = g32[i];
        iion = ms_point<float>(P, dt, v, h);
        g32[i] = h;
    } else if constexpr (KIND == MDX_KIND_TT) {
        double c[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) c[s] = u[s * ld + i];
        iion = tt_point<float>(P, dt, v, c, g32 + i, ld);
#pragma unroll
        for (int s = 0; s < 6; ++s) u[s * ld + i] = c[s];
    }
    const double src = (istim ? istim[i] : 0.0) - cm * iion;
    if constexpr (GATHER)
        put_gather(gather, i, v, src, gather.Vprev[i]);
    else
        out[i] = src;
}

// copy rows [row0, row0 + rows) of an FP64 SoA state block to FP32 or back
__global__ __launch_bounds__(256) void k_rows_to_f32(int64_t ld, int rows, const double *__restrict__ src,
                                                     float *__restrict__ dst)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ld * rows) return;
    dst[i] = (float)src[i];
}

__global__ __launch_bounds__(256) void k_rows_to_f64(int64_t ld, int rows, const float *__restrict__ src,
                                                     double *__restrict__ dst)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ld * rows) return;
    dst[i] = (double)src[i];
}

IonicParams pack(int kind, const double *params)
{
    IonicParams p{};
    int np = ionic_nparams(kind);
    for (int i = 0; i < np; ++i) p.v[i] = params[i];
    return p;
}

}  // namespace

int ionic_nstates(int kind) { return kind == 1 ? 1 : kind == 2 ? TT_NS : kind == 3 ? CRN_NS : 0; }
int ionic_nparams(int kind) { return kind == 1 ? MS_NP : kind == 2 ? TT_NP : kind == 3 ? CRN_NP : 0; }

void ionic_defaults(int kind, double *params)
{
    static const double ms[MS_NP] = {0.3, 6.0, 120.0, 150.0, 0.13, -80.0, 100.0};
    static const double tt[TT_NP] = {14.838, 5.405, 0.073, 0.153,  0.392,  3.98e-5,
                                     2.9e-4, 5.92e-4, 0.1238, 0.0146, 2.724, 1000.0};
    if (kind == 1)
        for (int i = 0; i < MS_NP; ++i) params[i] = ms[i];
    if (kind == 2)
        for (int i = 0; i < TT_NP; ++i) params[i] = tt[i];
    static const double crn_p[CRN_NP] = {7.8,     0.09,     0.1652,     0.029411765, 0.12941176,
                                         0.12375, 6.744375e-4, 1.131e-3, 0.59933874,  1600.0,
                                         0.275,   0.005,    1.0};
    if (kind == 3)
        for (int i = 0; i < CRN_NP; ++i) params[i] = crn_p[i];
}

void launch_ionic_init(hipStream_t s, int kind, const double *params, int64_t n, int64_t ld,
                       double *V, double *Vprev, double *u, const int32_t *tile_real)
{
    IonicParams P = pack(kind, params);
    dim3 grid((unsigned)((ld + 255) / 256)), block(256);
    if (kind == 1)
        hipLaunchKernelGGL(k_ionic_init<MDX_KIND_MS>, grid, block, 0, s, P, n, ld, V, Vprev, u, tile_real);
    else if (kind == 2)
        hipLaunchKernelGGL(k_ionic_init<MDX_KIND_TT>, grid, block, 0, s, P, n, ld, V, Vprev, u, tile_real);
    else if (kind == 3)
        hipLaunchKernelGGL(k_ionic_init<MDX_KIND_CRN>, grid, block, 0, s, P, n, ld, V, Vprev, u, tile_real);
    else
        hipLaunchKernelGGL(k_ionic_init<MDX_KIND_NONE>, grid, block, 0, s, P, n, ld, V, Vprev, u, tile_real);
}

void launch_ionic_step(hipStream_t s, int kind, const double *params, int64_t n, int64_t ld,
                       double dt, double cm, const double *V, double *u, const double *istim,
                       double *out, int raw, const int32_t *tile_real, const int32_t *guard,
                       const StepTimes &times, const GatherOut &gather)
{
    if (n <= 0) return;
    IonicParams P = pack(kind, params);
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
    void (*k)(IonicParams, int64_t, int64_t, double, double, const double *, double *, const double *,
              double *, int, const int32_t *, const int32_t *, StepTimes, GatherOut);
    const bool gv = gather.gv != nullptr;
    if (kind == 1)
        k = gv ? k_ionic_step<MDX_KIND_MS, true> : k_ionic_step<MDX_KIND_MS, false>;
    else if (kind == 2)
        k = gv ? k_ionic_step<MDX_KIND_TT, true> : k_ionic_step<MDX_KIND_TT, false>;
    else if (kind == 3)
        k = gv ? k_ionic_step<MDX_KIND_CRN, true> : k_ionic_step<MDX_KIND_CRN, false>;
    else
        k = gv ? k_ionic_step<MDX_KIND_NONE, true> : k_ionic_step<MDX_KIND_NONE, false>;
    hipLaunchKernelGGL(k, grid, block, 0, s, P, n, ld, dt, cm, V, u, istim, out, raw, tile_real, guard,
                       times, gather);
}

int ionic_gate_rows(int kind) { return kind == 1 ? 1 : kind == 2 ? 12 : 0; }
int ionic_gate_row0(int kind) { return kind == 1 ? 0 : kind == 2 ? 6 : 0; }

void launch_ionic_step_mixed(hipStream_t s, int kind, const double *params, int64_t n, int64_t ld,
                             double dt, double cm, const double *V, double *u, float *g32,
                             const double *istim, double *out, const int32_t *tile_real,
                             const int32_t *guard, const StepTimes &times, const GatherOut &gather)
{
    if (n <= 0) return;
    IonicParams P = pack(kind, params);
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
    void (*k)(IonicParams, int64_t, int64_t, double, double, const double *, double *, float *,
              const double *, double *, const int32_t *, const int32_t *, StepTimes, GatherOut);
    const bool gv = gather.gv != nullptr;
    if (kind == 1)
        k = gv ? k_ionic_step_mixed<MDX_KIND_MS, true> : k_ionic_step_mixed<MDX_KIND_MS, false>;
    else if (kind == 2)
        k = gv ? k_ionic_step_mixed<MDX_KIND_TT, true> : k_ionic_step_mixed<MDX_KIND_TT, false>;
    else
        k = gv ? k_ionic_step_mixed<MDX_KIND_NONE, true> : k_ionic_step_mixed<MDX_KIND_NONE, false>;
    hipLaunchKernelGGL(k, grid, block, 0, s, P, n, ld, dt, cm, V, u, g32, istim, out, tile_real, guard,
                       times, gather);
}

void launch_gates_to_f32(hipStream_t s, int kind, int64_t ld, const double *u, float *g32)
{
    const int rows = ionic_gate_rows(kind);
    if (rows == 0) return;
    const int64_t cnt = ld * rows;
    hipLaunchKernelGGL(k_rows_to_f32, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, ld, rows,
                       u + (int64_t)ionic_gate_row0(kind) * ld, g32);
}

void launch_gates_to_f64(hipStream_t s, int kind, int64_t ld, const float *g32, double *u)
{
    const int rows = ionic_gate_rows(kind);
    if (rows == 0) return;
    const int64_t cnt = ld * rows;
    hipLaunchKernelGGL(k_rows_to_f64, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, ld, rows,
                       g32, u + (int64_t)ionic_gate_row0(kind) * ld);
}

}  // namespace mdx
