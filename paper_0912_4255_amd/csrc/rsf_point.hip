// 2F at continuous parameters and its gradient (project addition on top of
// paper Sec. III.A.2): for every candidate theta = (f, f^(1), ..., f^(s),
// alpha, delta) at spindown order s = 1..3 (followed by the orbit (a_p, P_b,
// t_asc) for a source in a circular binary orbit) the resampled series of the
// candidate's own sky is recomputed on the fly
// (never stored) and reduced to
//   F_a = sum_k y^a_k exp(-2 pi i (f - f_het) t_b^k),   F_b likewise,
//   A', B', C'  (masked antenna sums),
// plus, for the gradient, the derivatives of all five with respect to
// theta, following every dependence of the resampling chain:
//   * f:     d/df exp(-2 pi i (f - f_het) t_b) = -2 pi i t_b (...);
//   * f^(j): Phi_s = 2 pi sum_j f^(j) (T^(j+1)/(j+1)! + t_m T^j/j!)  (eq. eq4pt1),
//            which at s = 1 is pi fdot (t_b^2 - t_m^2) with T = t_b - t_m;
//   * sky:   t_m(tau) = n0 . r_d(tau) (eq. eq4pt2); the inversion of eq. eq21
//            gives dT/dtheta = -(dt_m/dtheta)/(1 + dt_m/dt); the
//            interpolated series changes through the kernel derivative
//            w'(u - p) dT/dtheta / dt and through the heterodyne correction
//            dz_p/dtheta = -2 pi i f_het (dt_m/dtheta)(t_p) z_p (eq. absorb);
//            the beam patterns change through p, q(alpha, delta) and T; the
//            spindown phase through T at fixed t_b:
//            dPhi_s/dT = 2 pi t_m sum_j f^(j) T^(j-1)/(j-1)!;
//   * orbit: the inversion targets t_b + R(tau_e) (tau_e = t_start + t_b on
//            the emission grid), so dT/dtheta_o = (dR/dtheta_o)/(1 + dt_m/dt);
//            t_m is replaced by the total delay d = t_m - R(tau_e) (equal to
//            t_b - T), and at a detector sample p the correction's delay
//            d_p = t_m(t_p) - R(tau_e,p) with tau_e,p + R(tau_e,p) = tau_p +
//            t_m(t_p) changes by -(dR/dtheta_o)/(1 + R') for the orbit and by
//            (dt_m/dtheta)/(1 + R') for the sky, R' = dR/dtau at tau_e,p.
// Two kernels: rsf_point_run_k interpolates the timing chain along runs of 256
// samples and carries every ordinary call; rsf_point_k evaluates it per sample.
// Each block accumulates FP64 partial sums over up to 128 rows of 64 samples;
// rsf_point_reduce_k sums the blocks of a candidate in a fixed order and
// forms 2F (eq. eq6) and the vector-Jacobian product g * d2F/dtheta.
#include <climits>

#include "rsf_chain.h"
#include "rsf_launch.h"

namespace rsf {

namespace {
constexpr int kTileB = 64;
constexpr int kThreads = 256;
constexpr int kWinMax = kTileB + kMaxTaps + 8;

// partial-sum slots at spindown order ORDER: NP = 1 + ORDER + NS parameters,
// the last NS of which (alpha, delta, and a_p, P_b, t_asc for a binary
// source) move the resampled times and hence also A', B', C'
template <int ORDER, bool BIN>
struct Slots {
    static constexpr int NS = BIN ? 5 : 2;
    static constexpr int NP = 1 + ORDER + NS;
    static constexpr int FA = 0, FB = 2, A = 4, B = 5, C = 6;
    static constexpr int DFA = 7;             // NP parameters x (re, im)
    static constexpr int DFB = DFA + 2 * NP;
    static constexpr int DA = DFB + 2 * NP;   // NS parameters each
    static constexpr int DB = DA + NS;
    static constexpr int DC = DB + NS;
    static constexpr int USED = DC + NS;
};
static_assert(Slots<3, true>::USED <= kPointSums, "partial-sum stride too small");

// R(tau_e) of a circular orbit, with cos of its angle for the derivatives
__device__ __forceinline__ double orbit_delay(const BinaryOrbit& b, double tau_e, double& s_phi, double& c_phi) {
    const double cyc = (tau_e - b.t_asc) / b.p_orb;
    sincos(2.0 * kPi * (cyc - floor(cyc)), &s_phi, &c_phi);
    return b.a_p * s_phi;
}

// tau_e with tau_e + R(tau_e) = tau by two Newton steps from tau - R(tau):
// the start is off by at most max R' times max R (at most 1e-2 a_p), and each
// step squares the error times (2 pi / P_b)^2 a_p / 2, so two steps reach
// rounding for every admitted orbit.  The angle's sin and cos at the result
// come from those of the last evaluation turned by the last step (first order).
__device__ __forceinline__ double emission_newton(const BinaryOrbit& b, double tau, double& s_phi, double& c_phi) {
    const double w = 2.0 * kPi / b.p_orb;
    double te = tau - orbit_delay(b, tau, s_phi, c_phi);
    double r = orbit_delay(b, te, s_phi, c_phi);
    te -= (te + r - tau) / (1.0 + b.a_p * w * c_phi);
    r = orbit_delay(b, te, s_phi, c_phi);
    const double d = (te + r - tau) / (1.0 + b.a_p * w * c_phi);
    te -= d;
    const double s = s_phi - c_phi * (w * d), c = c_phi + s_phi * (w * d);
    s_phi = s;
    c_phi = c;
    return te;
}

// dR/d(a_p, P_b, t_asc) at tau_e from the angle's sin and cos
__device__ __forceinline__ void orbit_partials(const BinaryOrbit& b, double tau_e, double s_phi, double c_phi,
                                               double* dR) {
    const double w = 2.0 * kPi / b.p_orb;
    dR[0] = s_phi;
    dR[1] = -b.a_p * c_phi * w * (tau_e - b.t_asc) / b.p_orb;
    dR[2] = -b.a_p * c_phi * w;
}

// 1/j! for the spindown terms
__device__ constexpr double kInvFact[5] = {1.0, 1.0, 0.5, 1.0 / 6.0, 1.0 / 24.0};

struct Orbit {
    double3 r;       // r_d / c (s)
    double3 v;       // v_d / c
    double sl, cl;   // orbital angle (the orbital part of r is AU/c (cl, ceps sl, seps sl))
    double sth, cth;
};

__device__ __forceinline__ Orbit orbit_at(double tau, const EphDev& e, const DetDev& d) {
    const double lam = e.lambda0 + 2.0 * kPi * frac_rev(tau * e.inv_p_orb);
    const double th = e.theta0 + 2.0 * kPi * frac_rev(tau * e.inv_p_sid) + d.lon;
    double sl, cl, st, ct;
    sincos(lam, &sl, &cl);
    sincos(th, &st, &ct);
    const double wo = 2.0 * kPi * e.inv_p_orb, ws = 2.0 * kPi * e.inv_p_sid;
    Orbit o;
    o.r = make_double3(e.au_c * cl + e.re_c * d.clat * ct, e.au_c * e.ceps * sl + e.re_c * d.clat * st,
                       e.au_c * e.seps * sl + e.re_c * d.slat);
    o.v = make_double3(-e.au_c * wo * sl - e.re_c * ws * d.clat * st, e.au_c * wo * e.ceps * cl + e.re_c * ws * d.clat * ct,
                       e.au_c * wo * e.seps * cl);
    o.sl = sl;
    o.cl = cl;
    o.sth = st;
    o.cth = ct;
    return o;
}

__device__ __forceinline__ double dot3(double3 a, double3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }

// sin and cos of a small angle by their Taylor series through a^11 and
// a^10; for |a| <= 0.3 the first omitted terms are below 2e-15.
__device__ __forceinline__ void small_sincos(double a, double& s, double& c) {
    const double a2 = a * a;
    s = a * (1.0 - a2 * (1.0 / 6.0) *
                       (1.0 - a2 * (1.0 / 20.0) *
                                  (1.0 - a2 * (1.0 / 42.0) * (1.0 - a2 * (1.0 / 72.0) * (1.0 - a2 * (1.0 / 110.0))))));
    c = 1.0 - a2 * 0.5 *
                  (1.0 - a2 * (1.0 / 12.0) *
                             (1.0 - a2 * (1.0 / 30.0) * (1.0 - a2 * (1.0 / 56.0) * (1.0 - a2 * (1.0 / 90.0)))));
}

// (sin, cos) of x + a from those of x and a
__device__ __forceinline__ void rot_add(double sx, double cx, double sa, double ca, double& s, double& c) {
    s = sx * ca + cx * sa;
    c = cx * ca - sx * sa;
}

// Orbital and Greenwich sidereal angles at the first sample of the current
// run of a wave, as (sin, cos) pairs.  A wave's runs start 256 samples apart,
// so the pairs advance by a fixed rotation; a sample at tau_run + delta turns
// them by the small angles w delta, with |delta| <= 63 dt + max|t_m| (the
// host admits dt up to 55 s, which keeps w_sid |delta| below 0.3).
struct RunAngles {
    double sl, cl, sg, cg;
};

// The orbit of detector d at tau_run + delta.
__device__ __forceinline__ Orbit orbit_from(const RunAngles& ra, double delta, const EphDev& e, const DetDev& d,
                                            double wo, double ws) {
    double sa, ca, sb, cb, sl, cl, sg, cg, st, ct;
    small_sincos(wo * delta, sa, ca);
    small_sincos(ws * delta, sb, cb);
    rot_add(ra.sl, ra.cl, sa, ca, sl, cl);
    rot_add(ra.sg, ra.cg, sb, cb, sg, cg);
    rot_add(sg, cg, d.slon, d.clon, st, ct);  // local sidereal angle
    Orbit o;
    o.r = make_double3(e.au_c * cl + e.re_c * d.clat * ct, e.au_c * e.ceps * sl + e.re_c * d.clat * st,
                       e.au_c * e.seps * sl + e.re_c * d.slat);
    o.v = make_double3(-e.au_c * wo * sl - e.re_c * ws * d.clat * st, e.au_c * wo * e.ceps * cl + e.re_c * ws * d.clat * ct,
                       e.au_c * wo * e.seps * cl);
    o.sl = sl;
    o.cl = cl;
    o.sth = st;
    o.cth = ct;
    return o;
}

// m . r_d / c and its first three time derivatives at the orbit o (each
// part moves on a circle, so its second derivative is -w^2 times the
// position and the third -w^2 times the velocity); rez = R_E sin(lat) / c.
__device__ __forceinline__ RoemerD project(const Orbit& o, double3 m, const EphDev& e, double wo2, double ws2,
                                           double rez) {
    RoemerD q;
    q.tm = dot3(m, o.r);
    q.d1 = dot3(m, o.v);
    const double my = m.y * e.ceps + m.z * e.seps;
    const double pro = e.au_c * (m.x * o.cl + my * o.sl);
    const double pvo = sqrt(wo2) * e.au_c * (-m.x * o.sl + my * o.cl);
    const double prr = q.tm - pro - m.z * rez, pvr = q.d1 - pvo;
    q.d2 = -wo2 * pro - ws2 * prr;
    q.d3 = -wo2 * pvo - ws2 * pvr;
    return q;
}



// Interpolation weight w(x) and w'(x) (Lanczos-W or the periodic Dirichlet
// kernel of length n written as sinc(x) g(pi x / n)); sx, cx = sin/cos(pi x).
template <bool GRAD>
__device__ __forceinline__ void kernel_w(const InterpDev& ip, float x, float sx, float cx, float& w, float& dw) {
    const int W = ip.taps;
    float s0, ds0;
    sinc_d(x, sx, cx, s0, ds0);
    if (ip.kernel == 0) {
        if (fabsf(x) >= 0.5f * (float)W) {
            w = 0.f;
            dw = 0.f;
            return;
        }
        const float v = 2.f * x / (float)W;
        float s1, ds1;
        const float sv = __builtin_amdgcn_sinf(0.5f * v), cv = __builtin_amdgcn_cosf(0.5f * v);  // revolutions
        sinc_d(v, sv, cv, s1, ds1);
        w = s0 * s1;
        if (GRAD) dw = ds0 * s1 + s0 * ds1 * (2.f / (float)W);
    } else {
        const float y = x * (kPiF / (float)ip.n);
        float g, dg;
        if (fabsf(y) < 0.01f) {
            const float y2 = y * y;
            if (ip.n_odd) {  // y / sin(y)
                g = 1.f + y2 / 6.f + 7.f * y2 * y2 / 360.f;
                dg = y / 3.f + 7.f * y * y2 / 90.f;
            } else {         // y / tan(y)
                g = 1.f - y2 / 3.f - y2 * y2 / 45.f;
                dg = -2.f * y / 3.f - 4.f * y * y2 / 45.f;
            }
        } else {
            float sy, cy;
            sincosf(y, &sy, &cy);
            if (ip.n_odd) {
                g = y / sy;
                dg = 1.f / sy - y * cy / (sy * sy);
            } else {
                g = y * cy / sy;
                dg = cy / sy - y / (sy * sy);
            }
        }
        w = s0 * g;
        if (GRAD) dw = ds0 * g + s0 * dg * (kPiF / (float)ip.n);
    }
}

// The sky's unit vector n0, its derivatives, and the polarisation basis
// (p, q) with the derivatives the gradient needs.
struct SkyGeom {
    double3 n0, n0a, n0d, pp, qq, pa, qa, qd;
};

// The timing chain of one resampled sample (eqs. eq4pt2, eq21 and the beam
// patterns of eq2, eq3), and for the gradient its sky (and orbit)
// derivatives.
struct ChainOut {
    double T1;                   // fixed-point iterate of T, the window's expansion point
    RoemerD x0, xa, xd;          // n0.r, n0_alpha.r, n0_delta.r and their time derivatives at T1
    double T, av, bv, dTa, dTd, daa, dad, dba, dbd;
    double dTo[3], dao[3], dbo[3];
};

// The chain at t_b = tb, a sample dl0 seconds after the first sample of its
// run (whose orbital and sidereal angles are ra): one fixed-point step and one
// Newton step of the inversion (residual below 1e-12 s), then the beam
// patterns at T.
template <bool GRAD, bool BIN>
__device__ __forceinline__ ChainOut chain_at(const PointArgs& A, const DetDev& D, const RunAngles& ra, double dl0,
                                             double tb, const SkyGeom& g, const BinaryOrbit& bo, double wo,
                                             double w_sid) {
    const double3 n0 = g.n0, n0a = g.n0a, n0d = g.n0d, pp = g.pp, qq = g.qq, pa = g.pa, qa = g.qa, qd = g.qd;
    ChainOut c{};
    // eq. eq21: one fixed-point step and one Newton step (residual below 1e-12 s)
    // a binary source's grid is regular in emission time: the
    // target is t_b + R(t_start + t_b)
    double tgt = tb, dRk[3] = {0.0, 0.0, 0.0};
    if constexpr (BIN) {
        double sp, cp;
        const double te = A.t_start + tb;
        tgt = tb + orbit_delay(bo, te, sp, cp);
        if (GRAD) orbit_partials(bo, te, sp, cp, dRk);
    }
    const double dl = dl0 + (BIN ? tgt - tb : 0.0);  // offset from the run's first sample
    const double tm0 = dot3(n0, orbit_from(ra, dl, A.eph, D, wo, w_sid).r);
    c.T1 = tgt - tm0;
    const Orbit o1 = orbit_from(ra, dl - tm0, A.eph, D, wo, w_sid);
    {
        const double wo2 = 4.0 * kPi * kPi * A.eph.inv_p_orb * A.eph.inv_p_orb;
        const double ws2 = w_sid * w_sid;
        const double rez = A.eph.re_c * D.slat;
        c.x0 = project(o1, n0, A.eph, wo2, ws2, rez);
        if (GRAD) {
            c.xa = project(o1, n0a, A.eph, wo2, ws2, rez);
            c.xd = project(o1, n0d, A.eph, wo2, ws2, rez);
        }
    }
    const double dT = -(c.T1 + dot3(n0, o1.r) - tgt) / (1.0 + dot3(n0, o1.v));
    c.T = c.T1 + dT;
    // the orbit at T: positions moved by v dT, the sidereal angle turned by w_sid dT
    Orbit o = o1;
    o.r = make_double3(o1.r.x + o1.v.x * dT, o1.r.y + o1.v.y * dT, o1.r.z + o1.v.z * dT);
    {
        const double a = w_sid * dT;
        const double sa = a * (1.0 - a * a / 6.0), ca = 1.0 - 0.5 * a * a;
        o.sth = o1.sth * ca + o1.cth * sa;
        o.cth = o1.cth * ca - o1.sth * sa;
    }
    // arms at the local sidereal angle, and their rate of change
    const double3 eE = make_double3(-o.sth, o.cth, 0.0);
    const double3 eN = make_double3(-D.slat * o.cth, -D.slat * o.sth, D.clat);
    const double3 eEt = make_double3(-o.cth, -o.sth, 0.0);
    const double3 eNt = make_double3(D.slat * o.sth, -D.slat * o.cth, 0.0);
    const double3 uu = make_double3(D.cgu * eE.x + D.sgu * eN.x, D.cgu * eE.y + D.sgu * eN.y,
                                    D.cgu * eE.z + D.sgu * eN.z);
    const double3 vv = make_double3(D.cgv * eE.x + D.sgv * eN.x, D.cgv * eE.y + D.sgv * eN.y,
                                    D.cgv * eE.z + D.sgv * eN.z);
    const double up = dot3(uu, pp), uq = dot3(uu, qq), vp = dot3(vv, pp), vq = dot3(vv, qq);
    c.av = 0.5 * (up * up - uq * uq - vp * vp + vq * vq);
    c.bv = up * uq - vp * vq;
    if (GRAD) {
        const double tmdot = dot3(n0, o.v);
        c.dTa = -dot3(n0a, o.r) / (1.0 + tmdot);
        c.dTd = -dot3(n0d, o.r) / (1.0 + tmdot);
        const double3 ut = make_double3(D.cgu * eEt.x + D.sgu * eNt.x, D.cgu * eEt.y + D.sgu * eNt.y, 0.0);
        const double3 vt = make_double3(D.cgv * eEt.x + D.sgv * eNt.x, D.cgv * eEt.y + D.sgv * eNt.y, 0.0);
        // d/dT through the sidereal rotation (per second)
        const double upt = dot3(ut, pp) * w_sid, uqt = dot3(ut, qq) * w_sid;
        const double vpt = dot3(vt, pp) * w_sid, vqt = dot3(vt, qq) * w_sid;
        const double adT = up * upt - uq * uqt - vp * vpt + vq * vqt;
        const double bdT = upt * uq + up * uqt - vpt * vq - vp * vqt;
        // d/dalpha, d/ddelta at fixed T through p and q
        const double upa = dot3(uu, pa), uqa = dot3(uu, qa), vpa = dot3(vv, pa), vqa = dot3(vv, qa);
        const double uqd = dot3(uu, qd), vqd = dot3(vv, qd);
        c.daa = up * upa - uq * uqa - vp * vpa + vq * vqa + adT * c.dTa;
        c.dba = upa * uq + up * uqa - vpa * vq - vp * vqa + bdT * c.dTa;
        c.dad = -uq * uqd + vq * vqd + adT * c.dTd;
        c.dbd = up * uqd - vp * vqd + bdT * c.dTd;
        if constexpr (BIN) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                c.dTo[i] = dRk[i] / (1.0 + tmdot);
                c.dao[i] = adT * c.dTo[i];
                c.dbo[i] = bdT * c.dTo[i];
            }
        }
    }
    return c;
}

}  // namespace

// The sums of V values over the wave, value i in lane (i and the lanes that
// share its upper bits) of the result: each step hands half of the values to the
// lane across and keeps the other half, so V values take about V exchanges in
// place of 6 V.  Returns value `lane >> (6 - LOG2)` (V <= 2^LOG2), a fixed
// order of additions.
template <int LOG2, int V>
__device__ __forceinline__ double wave_sums(const double (&acc)[V], int lane) {
    constexpr int N = 1 << LOG2;
    static_assert(V <= N, "more values than slots");
    double v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = i < V ? acc[i < V ? i : 0] : 0.0;
#pragma unroll
    for (int st = 0; st < LOG2; ++st) {
        const int half = N >> (st + 1), off = 32 >> st;
        const bool up = lane & off;
#pragma unroll
        for (int i = 0; i < half; ++i) {
            const double keep = up ? v[i + half] : v[i], give = up ? v[i] : v[i + half];
            v[i] = keep + __shfl_xor(give, off);
        }
    }
#pragma unroll
    for (int off = 32 >> LOG2; off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off);
    return v[0];
}

// The point search's runs: 256 samples (four rows of 64).
constexpr int kRunRows = 4;
constexpr int kRunLen = kRunRows * kTileB;
struct PointRun {
    static constexpr double mid = 0.5 * (kRunLen - 1), half = 146.0, p = 138.5, q = 85.5;
};
constexpr double kRunMid = PointRun::mid;
constexpr int kRunsMax = 8 * 4;  // runs of a workgroup
// window of a run's rows: 64 samples and their compression (104 - W slots a
// row, as the general kernel stages), and the taps
constexpr int kRunWin = 416;

__device__ __forceinline__ bool orbit_interpolates(const BinaryOrbit& b, double dt) {
    return orbit_slow(b, PointRun::half * dt, kDelayErr);
}

// Per run: quartics in s of the NQ quantities V = d / dt, a, b (and, for the
// gradient, dT, da, db of the NS parameters that move T); the window's delay in
// cycles, f_het d, as a quartic in x = (detector sample) - u_c; and what the
// derivatives need beside them (below).
template <bool GRAD, int NS>
struct RunVals {
    static constexpr int NQ = GRAD ? 3 + 3 * NS : 3;
    double poly[NQ][5];
    double het[5], u_c;
    double G[3];                     // 1 / (1 - V'(s)) to second order
    double psi[GRAD ? NS : 1][3];    // see rsf_point_run_k
    double vn[5];                    // V at the nodes
    int gap, pad;                    // gap_state of the run
};

// The binary gradient's 50 to 58 FP64 partial sums do not fit beside the rest
// at two waves per SIMD; at one wave per SIMD its spills go to the
// accumulation registers instead of scratch memory.
// Takes the candidates that rsf_point_run_k leaves: sampling intervals too long
// for its interpolated chain, or an orbit too fast for it.
template <bool GRAD, int ORDER, bool BIN>
__global__ __launch_bounds__(kThreads, (BIN && GRAD) ? 1 : 2) void rsf_point_k(PointArgs A) {
    using SL = Slots<ORDER, BIN>;
    constexpr int NP = SL::NP;
    constexpr int S_FA = SL::FA, S_FB = SL::FB, S_A = SL::A, S_B = SL::B, S_C = SL::C;
    constexpr int S_DFA = SL::DFA, S_DFB = SL::DFB, S_DA = SL::DA, S_DB = SL::DB, S_DC = SL::DC;
    constexpr int S_USED = SL::USED;
    constexpr int S_SKY = 2 * (1 + ORDER);  // offset of (alpha, delta) within S_DFA / S_DFB
    __shared__ float4 win[4][kWinMax];  // z (re, im), 2 pi f_het dd_p/dalpha, 2 pi f_het dd_p/ddelta
    __shared__ float4 wino[4][(BIN && GRAD) ? kWinMax : 1];  // 2 pi f_het dd_p/d(a_p, P_b, t_asc)
    __shared__ double red[4][kPointSums];

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int cand = blockIdx.y;
    const double* th = A.theta + (int64_t)NP * cand;
    const double f = th[0], al = th[1 + ORDER], de = th[2 + ORDER];
    double fs[ORDER];  // f^(1) .. f^(ORDER)
#pragma unroll
    for (int i = 0; i < ORDER; ++i) fs[i] = th[1 + i];
    const double fd = fs[0];
    BinaryOrbit bo{};
    bool orbit_ok = true;
    if constexpr (BIN) {
        const BinaryOrbit given{th[3 + ORDER], th[4 + ORDER], th[5 + ORDER]};
        orbit_ok = orbit_admitted(given);
        bo = orbit_or_none(given);
        if (A.run && orbit_ok && orbit_interpolates(bo, A.dt)) return;
    }
    double sa, ca, sd, cd;
    sincos(al, &sa, &ca);
    sincos(de, &sd, &cd);
    const double3 n0 = make_double3(cd * ca, cd * sa, sd);
    const double3 n0a = make_double3(-cd * sa, cd * ca, 0.0);
    const double3 n0d = make_double3(-sd * ca, -sd * sa, cd);
    const double3 pp = make_double3(-sa, ca, 0.0);
    const double3 qq = make_double3(-sd * ca, -sd * sa, cd);
    const double3 pa = make_double3(-ca, -sa, 0.0);          // dp/dalpha (dp/ddelta = 0)
    const double3 qa = make_double3(sd * sa, -sd * ca, 0.0);  // dq/dalpha
    const double3 qd = make_double3(-cd * ca, -cd * sa, -sd); // dq/ddelta
    const SkyGeom geo{n0, n0a, n0d, pp, qq, pa, qa, qd};
    const double w_sid = 2.0 * kPi * A.eph.inv_p_sid;
    const int W = A.ip.taps;
    const int hw = W / 2;
    // Dirichlet weights by their small-argument series when pi x / n < 0.01 on every tap
    const float pin = kPiF / (float)A.ip.n;
    const bool dir_series = A.ip.kernel == 1 && pin * (float)(hw + 1) < 0.01f;
    // ... and when pi x / n < 2.9e-4 on every tap, g = 1 and g' pi / n = 0 to
    // FP32 precision: the weights are sinc(x) and its derivative
    const bool dir_flat = A.ip.kernel == 1 && pin * (float)(hw + 1) < 2.9e-4f;

    double acc[S_USED];
#pragma unroll
    for (int i = 0; i < S_USED; ++i) acc[i] = 0.0;
    bool overflow = false;

    // angles at this wave's first run, and the rotation to the next run
    const double wo = 2.0 * kPi * A.eph.inv_p_orb;
    RunAngles ra;
    double s_dl, c_dl, s_dg, c_dg;
    {
        const int64_t k_first = ((int64_t)blockIdx.x * A.rows * 4 + wave) * kTileB;
        const double tau0 = A.t_start + (double)k_first * A.dt;
        sincos(A.eph.lambda0 + 2.0 * kPi * frac_rev(tau0 * A.eph.inv_p_orb), &ra.sl, &ra.cl);
        sincos(A.eph.theta0 + 2.0 * kPi * frac_rev(tau0 * A.eph.inv_p_sid), &ra.sg, &ra.cg);
        const double dtau = 4.0 * kTileB * A.dt;
        sincos(wo * dtau, &s_dl, &c_dl);
        sincos(w_sid * dtau, &s_dg, &c_dg);
    }

    {
        for (int r = 0; r < A.rows; ++r) {
            const int64_t row = ((int64_t)blockIdx.x * A.rows + r) * 4 + wave;
            const int64_t k = row * kTileB + lane;
            const bool valid = (row < A.P) && (k < A.n);
            const double tb = (double)k * A.dt;
            for (int X = 0; X < A.n_det; ++X) {
                const DetDev& D = A.det[X];
                int j = 0;
                float frac = 0.f;
                double T = tb, tm = 0.0;
                bool mk = false;
                ChainOut c{};
                double t_ref;
                RoemerD q0, qa{}, qd{};
                if (valid) {
                    c = chain_at<GRAD, BIN>(A, D, ra, (double)lane * A.dt, tb, geo, bo, wo, w_sid);
                    T = c.T;
                    tm = tb - T;
                }
                // expansion point of t_m (and of its sky derivatives) for the
                // window: the first valid lane's fixed-point iterate
                const uint64_t vmask = __ballot(valid);
                const int src = vmask ? __ffsll((long long)vmask) - 1 : 0;
                t_ref = readlane_d(c.T1, src);
                q0 = readlane_rd(c.x0, src);
                if (GRAD) {
                    qa = readlane_rd(c.xa, src);
                    qd = readlane_rd(c.xd, src);
                }
                if (valid) {
                    const double u = T / A.dt;
                    const double fl = floor(u);
                    j = (int)fl;
                    frac = (float)(u - fl);
                    const int64_t jn = (int64_t)floor(u + 0.5);
                    mk = (jn >= 0) && (jn < A.n) && !in_gap(A.gaps[X], A.n_gaps[X], jn);
                }
                const double av = c.av, bv = c.bv, dTa = c.dTa, dTd = c.dTd;
                const double daa = c.daa, dad = c.dad, dba = c.dba, dbd = c.dbd;
                const double* dTo = c.dTo;
                const double* dao = c.dao;
                const double* dbo = c.dbo;
                // detector-grid window of this run, heterodyne-corrected
                int jmin = valid ? j : INT_MAX;
                int jmax = valid ? j : INT_MIN;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    jmin = min(jmin, __shfl_xor(jmin, off));
                    jmax = max(jmax, __shfl_xor(jmax, off));
                }
                const bool any = jmin != INT_MAX;
                const int w0 = any ? jmin - hw + 1 : 0;
                const int wlen = any ? (jmax - jmin + W) : 0;
                const bool ok = wlen <= kWinMax;
                if (any && ok) {
                    for (int p = lane; p < wlen; p += 64) {
                        const int64_t jj = (int64_t)w0 + p;
                        float4 e = make_float4(0.f, 0.f, 0.f, 0.f);
                        float4 eo = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (jj >= 0 && jj < A.n) {
                            const float2 xv = A.x[X][jj];
                            const double dl = (double)jj * A.dt - t_ref;
                            double tmj = tm_expand(q0, dl);
                            double inv1r = 1.0;  // 1 / (1 + R') at this sample's emission time
                            if constexpr (BIN) {
                                // total delay d_p = t_m - R(tau_e), tau_e + R(tau_e) = tau_p + t_m
                                double sp, cp;
                                const double te = emission_newton(bo, A.t_start + (double)jj * A.dt + tmj, sp, cp);
                                tmj -= bo.a_p * sp;
                                if (GRAD) {
                                    inv1r = 1.0 / (1.0 + bo.a_p * cp * (2.0 * kPi / bo.p_orb));
                                    double dR[3];
                                    orbit_partials(bo, te, sp, cp, dR);
                                    const double k = -2.0 * kPi * A.f_het * inv1r;
                                    eo = make_float4((float)(k * dR[0]), (float)(k * dR[1]), (float)(k * dR[2]), 0.f);
                                }
                            }
                            const double cyc = A.f_het * tmj;
                            const float ph = (float)(cyc - rint(cyc));
                            const float s = __builtin_amdgcn_sinf(ph), c = __builtin_amdgcn_cosf(ph);  // revolutions
                            e.x = xv.x * c + xv.y * s;
                            e.y = xv.y * c - xv.x * s;
                            if (GRAD) {
                                e.z = (float)(2.0 * kPi * A.f_het * tm_expand(qa, dl) * inv1r);
                                e.w = (float)(2.0 * kPi * A.f_het * tm_expand(qd, dl) * inv1r);
                            }
                        }
                        win[wave][p] = e;
                        if constexpr (BIN && GRAD) wino[wave][p] = eo;
                    }
                }
                if (any && !ok) overflow = true;
                // the window is this wave's own: its LDS operations complete in
                // order, so a wave-level barrier suffices
                __builtin_amdgcn_wave_barrier();
                if (valid && ok) {
                    // interpolation (and derivative pieces)
                    const float sf = __builtin_amdgcn_sinf(0.5f * frac), cf = __builtin_amdgcn_cosf(0.5f * frac);
                    float2 zt = make_float2(0.f, 0.f), s1 = zt, sza = zt, szd = zt;
                    float2 szo[3] = {zt, zt, zt};
                    const int base = j - hw + 1 - w0;
                    for (int i = 1; i <= W; ++i) {
                        const float x = frac + (float)(hw - i);
                        const bool odd = (hw - i) & 1;
                        const float sx = odd ? -sf : sf, cx = odd ? -cf : cf;  // sin, cos of pi x
                        float w, dw = 0.f;
                        if (x == 0.f) {
                            w = 1.f;
                            dw = 0.f;
                        } else if (dir_flat) {
                            sinc_d(x, sx, cx, w, dw);
                        } else if (dir_series) {
                            // Dirichlet kernel of a long series: sinc(x) g(y), y = pi x / n
                            // small, g = y / tan(y) (n even) or y / sin(y) (n odd) as a series
                            float s0, ds0;
                            sinc_d(x, sx, cx, s0, ds0);
                            const float y = x * pin, y2 = y * y;
                            const float g = A.ip.n_odd ? 1.f + y2 * (1.f / 6.f + y2 * (7.f / 360.f))
                                                       : 1.f - y2 * (1.f / 3.f + y2 * (1.f / 45.f));
                            w = s0 * g;
                            if (GRAD) {
                                const float dg = A.ip.n_odd ? y * (1.f / 3.f + y2 * (7.f / 90.f))
                                                            : -y * (2.f / 3.f + y2 * (4.f / 45.f));
                                dw = ds0 * g + s0 * dg * pin;
                            }
                        } else {
                            kernel_w<GRAD>(A.ip, x, sx, cx, w, dw);
                        }
                        const float4 zz = win[wave][base + i - 1];
                        zt.x += w * zz.x;
                        zt.y += w * zz.y;
                        if (GRAD) {
                            s1.x += dw * zz.x;
                            s1.y += dw * zz.y;
                            sza.x += w * zz.z * zz.x;
                            sza.y += w * zz.z * zz.y;
                            szd.x += w * zz.w * zz.x;
                            szd.y += w * zz.w * zz.y;
                            if constexpr (BIN) {
                                const float4 oo = wino[wave][base + i - 1];
                                szo[0].x += w * oo.x * zz.x;
                                szo[0].y += w * oo.x * zz.y;
                                szo[1].x += w * oo.y * zz.x;
                                szo[1].y += w * oo.y * zz.y;
                                szo[2].x += w * oo.z * zz.x;
                                szo[2].y += w * oo.z * zz.y;
                            }
                        }
                    }
                    // total phase: spindown Phi_s and the Fourier kernel at f;
                    // us[j] = T^(j+2)/(j+2)! + t_m T^(j+1)/(j+1)! (cycles per unit f^(j+1))
                    double us[ORDER];
                    double cyc;
                    if constexpr (ORDER == 1) {
                        cyc = fd * 0.5 * (tb * tb - tm * tm) + (f - A.f_het) * tb;
                    } else {
                        double Tj = T;  // T^(j+1)
                        cyc = (f - A.f_het) * tb;
#pragma unroll
                        for (int i = 0; i < ORDER; ++i) {
                            us[i] = Tj * T * kInvFact[i + 2] + tm * Tj * kInvFact[i + 1];
                            cyc += fs[i] * us[i];
                            Tj *= T;
                        }
                    }
                    const float ph = (float)(cyc - rint(cyc));
                    const float s = __builtin_amdgcn_sinf(ph), c = __builtin_amdgcn_cosf(ph);  // revolutions
                    // ze = z~ exp(-2 pi i cyc)
                    const float zer = zt.x * c + zt.y * s, zei = zt.y * c - zt.x * s;
                    const double w = D.w;
                    acc[S_FA + 0] += w * av * zer;
                    acc[S_FA + 1] += w * av * zei;
                    acc[S_FB + 0] += w * bv * zer;
                    acc[S_FB + 1] += w * bv * zei;
                    if (mk) {
                        acc[S_A] += w * av * av;
                        acc[S_B] += w * bv * bv;
                        acc[S_C] += w * av * bv;
                    }
                    if (GRAD) {
                        // d/df: -2 pi i t_b ; d/df^(j): -2 pi i us[j-1]
                        // (at order 1: -i pi (t_b^2 - t_m^2))
                        const double cf_ = 2.0 * kPi * tb;
                        // (-i c) (x + i y) = c y - i c x
                        acc[S_DFA + 0] += w * av * cf_ * zei;
                        acc[S_DFA + 1] -= w * av * cf_ * zer;
                        acc[S_DFB + 0] += w * bv * cf_ * zei;
                        acc[S_DFB + 1] -= w * bv * cf_ * zer;
                        // dPhi_s/dT / (2 pi t_m) = sum_j f^(j) T^(j-1)/(j-1)!
                        double rate;
                        if constexpr (ORDER == 1) {
                            const double cfd = kPi * (tb * tb - tm * tm);
                            acc[S_DFA + 2] += w * av * cfd * zei;
                            acc[S_DFA + 3] -= w * av * cfd * zer;
                            acc[S_DFB + 2] += w * bv * cfd * zei;
                            acc[S_DFB + 3] -= w * bv * cfd * zer;
                            rate = fd;
                        } else {
                            double Tj = 1.0;
                            rate = 0.0;
#pragma unroll
                            for (int i = 0; i < ORDER; ++i) {
                                const double cu = 2.0 * kPi * us[i];
                                acc[S_DFA + 2 + 2 * i] += w * av * cu * zei;
                                acc[S_DFA + 3 + 2 * i] -= w * av * cu * zer;
                                acc[S_DFB + 2 + 2 * i] += w * bv * cu * zei;
                                acc[S_DFB + 3 + 2 * i] -= w * bv * cu * zer;
                                rate += fs[i] * Tj * kInvFact[i];
                                Tj *= T;
                            }
                        }
                        // sky: dz~/dth = s1 dT/dth / dt - i sz_th ; dPhi/dth = dPhi_s/dT dT/dth
                        const float dTa_u = (float)(dTa / A.dt), dTd_u = (float)(dTd / A.dt);
                        const float dpa = (float)(2.0 * kPi * rate * tm * dTa);
                        const float dpd = (float)(2.0 * kPi * rate * tm * dTd);
                        // dz~_alpha = (s1.x dTa_u + sza.y, s1.y dTa_u - sza.x)
                        const float dza_r = s1.x * dTa_u + sza.y, dza_i = s1.y * dTa_u - sza.x;
                        const float dzd_r = s1.x * dTd_u + szd.y, dzd_i = s1.y * dTd_u - szd.x;
                        // rotate by exp(-2 pi i cyc)
                        const float ea_r = dza_r * c + dza_i * s, ea_i = dza_i * c - dza_r * s;
                        const float ed_r = dzd_r * c + dzd_i * s, ed_i = dzd_i * c - dzd_r * s;
                        // d(a ze)/dth = da ze + a (dz~ e) + a ze (-i dPhi)
                        acc[S_DFA + S_SKY + 0] += w * (daa * zer + av * ea_r + av * dpa * zei);
                        acc[S_DFA + S_SKY + 1] += w * (daa * zei + av * ea_i - av * dpa * zer);
                        acc[S_DFA + S_SKY + 2] += w * (dad * zer + av * ed_r + av * dpd * zei);
                        acc[S_DFA + S_SKY + 3] += w * (dad * zei + av * ed_i - av * dpd * zer);
                        acc[S_DFB + S_SKY + 0] += w * (dba * zer + bv * ea_r + bv * dpa * zei);
                        acc[S_DFB + S_SKY + 1] += w * (dba * zei + bv * ea_i - bv * dpa * zer);
                        acc[S_DFB + S_SKY + 2] += w * (dbd * zer + bv * ed_r + bv * dpd * zei);
                        acc[S_DFB + S_SKY + 3] += w * (dbd * zei + bv * ed_i - bv * dpd * zer);
                        if (mk) {
                            acc[S_DA + 0] += w * 2.0 * av * daa;
                            acc[S_DA + 1] += w * 2.0 * av * dad;
                            acc[S_DB + 0] += w * 2.0 * bv * dba;
                            acc[S_DB + 1] += w * 2.0 * bv * dbd;
                            acc[S_DC + 0] += w * (daa * bv + av * dba);
                            acc[S_DC + 1] += w * (dad * bv + av * dbd);
                        }
                        if constexpr (BIN) {
                            // the orbit moves T like the sky does, through dT/dtheta_o
#pragma unroll
                            for (int i = 0; i < 3; ++i) {
                                const float dTo_u = (float)(dTo[i] / A.dt);
                                const float dpo = (float)(2.0 * kPi * rate * tm * dTo[i]);
                                const float dz_r = s1.x * dTo_u + szo[i].y, dz_i = s1.y * dTo_u - szo[i].x;
                                const float eo_r = dz_r * c + dz_i * s, eo_i = dz_i * c - dz_r * s;
                                acc[S_DFA + S_SKY + 4 + 2 * i] += w * (dao[i] * zer + av * eo_r + av * dpo * zei);
                                acc[S_DFA + S_SKY + 5 + 2 * i] += w * (dao[i] * zei + av * eo_i - av * dpo * zer);
                                acc[S_DFB + S_SKY + 4 + 2 * i] += w * (dbo[i] * zer + bv * eo_r + bv * dpo * zei);
                                acc[S_DFB + S_SKY + 5 + 2 * i] += w * (dbo[i] * zei + bv * eo_i - bv * dpo * zer);
                                if (mk) {
                                    acc[S_DA + 2 + i] += w * 2.0 * av * dao[i];
                                    acc[S_DB + 2 + i] += w * 2.0 * bv * dbo[i];
                                    acc[S_DC + 2 + i] += w * (dao[i] * bv + av * dbo[i]);
                                }
                            }
                        }
                    }
                } else if (valid && !ok) {
                    acc[S_FA] = __longlong_as_double(0x7ff8000000000000LL);
                }
                __builtin_amdgcn_wave_barrier();  // the next run rewrites this wave's window
            }
            rot_add(ra.sl, ra.cl, s_dl, c_dl, ra.sl, ra.cl);
            rot_add(ra.sg, ra.cg, s_dg, c_dg, ra.sg, ra.cg);
        }
    }
    if (overflow && lane == 0) atomicOr(A.flags, 2u);
    if (!orbit_ok) {
        // a refused orbit: NaN 2F and gradient for this candidate
        acc[S_FA] = __longlong_as_double(0x7ff8000000000000LL);
        if (threadIdx.x == 0) atomicOr(A.flags, 4u);
    }

    // block reduction in a fixed order
    // unrolled: a loop-indexed acc would live in scratch memory
    constexpr int nsum = GRAD ? S_USED : S_DFA;
#pragma unroll
    for (int i = 0; i < nsum; ++i) {
        double v = acc[i];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) red[wave][i] = v;
    }
    __syncthreads();
    if (threadIdx.x < nsum) {
        const int i = threadIdx.x;
        const double t = ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
        A.partials[((int64_t)cand * A.n_blocks + blockIdx.x) * kPointSums + i] = t;
    }
}

// 2F's partial sums (and the gradient's) with the interpolated timing chain.
// Per run of 256 samples and detector:
//   * the nodes of all the workgroup's runs are evaluated first, one per thread
//     (chain_at), and turned into quartics;
//   * the run's detector samples are heterodyne-corrected once into the wave's
//     window in LDS, the delay at a detector sample from its own quartic;
//   * every sample interpolates z~ with w, and for the gradient also the sums
//     with w' (s1) and with the kernel's first moment (m1 = sum w_p (p - u) z_p;
//     for an orbit the second, m2, too).  The heterodyne correction's derivative
//     is smooth over the window, so its sum is its value at u times z~ plus
//     its slope times m1 (plus half its curvature times m2):
//       dz~/dtheta = s1 dT/dt - i (2 pi f_het D z~ + psi m1 + chi m2 / 2),
//     D = (dd/dtheta at fixed T) = -dT (1 + dd/dT) = -dT G, since d(T; theta) =
//     t_b - T along the inversion; psi = 2 pi f_het dD/du, chi = 2 pi f_het
//     d2D/du2 in samples.  For an isolated source D's curvature (1e-10 s per
//     sample^2 on 500 s) is far below FP32.
//     For the Dirichlet kernel of a long series w = (-1)^m sin(pi f) / (pi x),
//     so z~, s1 and m1 are sums of (-1)^m z / x, (-1)^m z / x^2 and (-1)^m z; the
//     two taps next to u keep the series form near x = 0.
// What bounds it: vector issue.  128 candidates of 1,728,000 samples: 3.40 ms with
// the gradient and 1.78 ms without, against 9.33 and 5.35 ms for quadratics per
// 64 samples with the correction's derivatives per window sample and tap; 16
// binary candidates: 0.88 and 0.27 ms against 4.17 and 1.72 ms (every sample's
// chain and two Newton steps per window sample); one candidate of 21,600 samples
// at 4 s: 14.5 and 12.7 us against 202 and 145 us (three workgroups).
template <bool GRAD, int ORDER, bool BIN>
__global__ __launch_bounds__(kThreads, (BIN && GRAD) ? 2 : (GRAD ? 3 : 4)) void rsf_point_run_k(PointArgs A) {
    using SL = Slots<ORDER, BIN>;
    constexpr int NP = SL::NP, NS = SL::NS;
    constexpr int S_FA = SL::FA, S_FB = SL::FB, S_A = SL::A, S_B = SL::B, S_C = SL::C;
    constexpr int S_DFA = SL::DFA, S_DFB = SL::DFB, S_DA = SL::DA, S_DB = SL::DB, S_DC = SL::DC;
    constexpr int S_SKY = 2 * (1 + ORDER);  // offset of the parameters that move T within S_DFA / S_DFB
    constexpr int NSUM = GRAD ? SL::USED : S_DFA;
    constexpr int LOG2 = NSUM <= 8 ? 3 : NSUM <= 32 ? 5 : 6;
    using RV = RunVals<GRAD, NS>;
    constexpr int NQ = RV::NQ;
    __shared__ RV runs[kRunsMax];
    __shared__ float2 win[4][kRunWin];
    __shared__ double red[4][kPointSums];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cand = blockIdx.y;
    const double* th = A.theta + (int64_t)NP * cand;
    BinaryOrbit bo{};
    if constexpr (BIN) {
        bo = BinaryOrbit{th[3 + ORDER], th[4 + ORDER], th[5 + ORDER]};
        if (!orbit_admitted(bo) || !orbit_interpolates(bo, A.dt)) return;  // rsf_point_k's
    }
    const double f = th[0];
    double fs[ORDER];  // f^(1) .. f^(ORDER)
#pragma unroll
    for (int i = 0; i < ORDER; ++i) fs[i] = th[1 + i];
    const int W = A.ip.taps, hw = W / 2;
    const float pin = kPiF / (float)A.ip.n;
    const bool dir_series = A.ip.kernel == 1 && pin * (float)(hw + 1) < 0.01f;
    // pi x / n < 2.9e-4 on every tap: g = 1 and g' pi / n = 0 to FP32 precision
    const bool dir_flat = A.ip.kernel == 1 && pin * (float)(hw + 1) < 2.9e-4f;
    // rows of this workgroup: with one row per wave the four waves share a run
    const int n_runs = max(1, A.rows / kRunRows) * (A.rows >= kRunRows ? 4 : 1);
    const int64_t row_b = (int64_t)blockIdx.x * 4 * A.rows;  // first row

    double acc[NSUM];
#pragma unroll
    for (int i = 0; i < NSUM; ++i) acc[i] = 0.0;
    bool overflow = false;

    for (int X = 0; X < A.n_det; ++X) {
        const DetDev& D = A.det[X];
        // nodes
        __syncthreads();
        if (tid < 5 * n_runs) {
            const int rr = tid / 5, i = tid - 5 * rr;
            double sa, ca, sd, cd;
            sincos(th[1 + ORDER], &sa, &ca);
            sincos(th[2 + ORDER], &sd, &cd);
            SkyGeom geo;
            geo.n0 = make_double3(cd * ca, cd * sa, sd);
            geo.n0a = make_double3(-cd * sa, cd * ca, 0.0);
            geo.n0d = make_double3(-sd * ca, -sd * sa, cd);
            geo.pp = make_double3(-sa, ca, 0.0);
            geo.qq = geo.n0d;
            geo.pa = make_double3(-ca, -sa, 0.0);
            geo.qa = make_double3(sd * sa, -sd * ca, 0.0);
            geo.qd = make_double3(-cd * ca, -cd * sa, -sd);
            const double s = node_at<PointRun>(i);
            const double tb = ((double)((row_b + (int64_t)rr * kRunRows) * kTileB) + (kRunMid + s)) * A.dt;
            const double tau = A.t_start + tb;
            RunAngles ra;
            sincos(A.eph.lambda0 + 2.0 * kPi * frac_rev(tau * A.eph.inv_p_orb), &ra.sl, &ra.cl);
            sincos(A.eph.theta0 + 2.0 * kPi * frac_rev(tau * A.eph.inv_p_sid), &ra.sg, &ra.cg);
            const ChainOut c = chain_at<GRAD, BIN>(A, D, ra, 0.0, tb, geo, bo, 2.0 * kPi * A.eph.inv_p_orb,
                                                   2.0 * kPi * A.eph.inv_p_sid);
            RV& v = runs[rr];
            const double V = (tb - c.T) / A.dt;
            v.vn[i] = V;
            v.poly[0][i] = V;
            v.poly[1][i] = c.av;
            v.poly[2][i] = c.bv;
            if constexpr (GRAD) {
                v.poly[3][i] = c.dTa;
                v.poly[4][i] = c.dTd;
                v.poly[3 + NS][i] = c.daa;
                v.poly[4 + NS][i] = c.dad;
                v.poly[3 + 2 * NS][i] = c.dba;
                v.poly[4 + 2 * NS][i] = c.dbd;
                if constexpr (BIN) {
#pragma unroll
                    for (int o = 0; o < 3; ++o) {
                        v.poly[5 + o][i] = c.dTo[o];
                        v.poly[5 + NS + o][i] = c.dao[o];
                        v.poly[5 + 2 * NS + o][i] = c.dbo[o];
                    }
                }
            }
        }
        __syncthreads();
        // quartics, one quantity per thread; the window's delay is the last
        for (int e = tid; e < n_runs * (NQ + 1); e += kThreads) {
            const int rr = e / (NQ + 1), qi = e - rr * (NQ + 1);
            RV& v = runs[rr];
            if (qi < NQ) {
                to_quartic<PointRun>(v.poly[qi]);
            } else {
                const double uc = (double)((row_b + (int64_t)rr * kRunRows) * kTileB) + kRunMid - v.vn[2];
                window_delay<PointRun>(v.vn, A.f_het * A.dt, v.het);
                v.u_c = uc;
            }
        }
        __syncthreads();
        if (tid < n_runs) {
            RV& v = runs[tid];
            const double* V = v.poly[0];
            // G = 1 / (1 - V'): V' = V1 + 2 V2 s + 3 V3 s^2
            const double G = 1.0 / (1.0 - V[1]), G2 = G * G;
            v.G[0] = G;
            v.G[1] = 2.0 * V[2] * G2;
            v.G[2] = (3.0 * V[3] + 4.0 * V[2] * V[2] * G) * G2;
            if constexpr (GRAD) {
                const double k = -2.0 * kPi * A.f_het * G2;
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const double* t = v.poly[3 + i];
                    // psi = 2 pi f_het dD/du and its slope along the run, chi / 2
                    v.psi[i][0] = k * (t[1] + t[0] * (2.0 * V[2]) * G);
                    v.psi[i][1] = k * (2.0 * t[2] + 3.0 * t[1] * (2.0 * V[2]) + t[0] * (6.0 * V[3]));
                    v.psi[i][2] = k * t[2] * G;
                }
            }
            // gaps: does one start or end near the run's samples (nearest-sample
            // mask), or are all of them inside one?
            const double k0 = (double)((row_b + (int64_t)tid * kRunRows) * kTileB);
            const int64_t lo = (int64_t)floor(k0 - quartic(V, -kRunMid)) - 2;
            const int64_t hi = (int64_t)floor(k0 + (kRunLen - 1) - quartic(V, kRunMid)) + 3;
            v.gap = gap_state(A.gaps[X], A.n_gaps[X], lo, hi);
        }
        __syncthreads();

        for (int rr0 = 0; rr0 < n_runs; rr0 += 4) {
            const int rr = A.rows >= kRunRows ? wave * (n_runs / 4) + rr0 / 4 : 0;
            const int r0 = A.rows >= kRunRows ? 0 : wave, r1 = A.rows >= kRunRows ? kRunRows : wave + 1;
            const RV& v = runs[rr];
            const int64_t k_run = (row_b + (int64_t)rr * kRunRows) * kTileB;  // the run's first sample
            const int last = (int)min((int64_t)(r1 * kTileB), A.n - k_run) - 1;  // last valid index in the run
            if (last < r0 * kTileB) continue;
            // detector-grid window of these rows, heterodyne-corrected
            const double V0 = quartic(v.poly[0], (double)(r0 * kTileB) - kRunMid);
            const double V1 = quartic(v.poly[0], (double)last - kRunMid);
            const int64_t j0 = (int64_t)floor((double)(k_run + r0 * kTileB) - V0);
            const int64_t j1 = (int64_t)floor((double)(k_run + last) - V1);
            const int64_t w0 = j0 - hw + 1;
            const int64_t wlen64 = j1 - j0 + W;
            const bool ok = j1 >= j0 && wlen64 <= (r1 - r0) * (104 - W) + W;
            const int wlen = ok ? (int)wlen64 : 0;
            if (!ok) overflow = true;
            const float2* xs = A.x[X];
            const double xc = (double)w0 - v.u_c;
            for (int p0 = 0; p0 < wlen; p0 += 320) {
                float2 xv[5];
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const int p = p0 + 64 * q + lane;
                    const int64_t jj = w0 + p;
                    xv[q] = (p < wlen && jj >= 0 && jj < A.n) ? xs[jj] : make_float2(0.f, 0.f);
                }
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const int p = p0 + 64 * q + lane;
                    if (p0 + 64 * q < wlen) {
                        const double cyc = quartic(v.het, xc + (double)p);
                        const float ph = (float)(cyc - rint(cyc));
                        const float sn = __builtin_amdgcn_sinf(ph), cs = __builtin_amdgcn_cosf(ph);  // revolutions
                        if (p < wlen)
                            win[wave][p] = make_float2(xv[q].x * cs + xv[q].y * sn, xv[q].y * cs - xv[q].x * sn);
                    }
                }
            }
            // the window is this wave's own: its LDS operations complete in
            // order, so a wave-level barrier suffices
            __builtin_amdgcn_wave_barrier();
            for (int r = r0; r < r1; ++r) {
                const int l = r * kTileB + lane;
                if (l > last) continue;
                const int64_t k = k_run + l;
                const double s = (double)l - kRunMid;
                const double V = quartic(v.poly[0], s);
                const double u = (double)k - V, fl = floor(u);
                const float frac = (float)(u - fl);
                const int base = (int)((int64_t)fl - hw + 1 - w0);  // slot of tap 1
                if (!ok || base < 0 || base + W > wlen) {
                    overflow = true;
                    acc[S_FA] = __longlong_as_double(0x7ff8000000000000LL);
                    continue;
                }
                const float2* wz = win[wave] + base;
                float2 zt, s1 = make_float2(0.f, 0.f), m1 = s1, m2 = s1;
                const float sf = __builtin_amdgcn_sinf(0.5f * frac), cf = __builtin_amdgcn_cosf(0.5f * frac);
                if (dir_flat) {
                    // taps hw (x = frac) and hw + 1 (x = frac - 1)
                    float w0_, dw0, w1_, dw1;
                    const float x1 = frac - 1.f;
                    sinc_d(frac, sf, cf, w0_, dw0);
                    sinc_d(x1, -sf, -cf, w1_, dw1);
                    const float2 za = wz[hw - 1], zb = wz[hw];
                    float2 a1 = make_float2(0.f, 0.f), a2 = a1, a0 = a1, ax = a1;
                    // taps hw - m (x = frac + m, sign (-1)^m) and hw + 1 + m (x = frac - 1 - m, sign -(-1)^m)
                    auto pair = [&](int m, float sg) {
                        const float2 zl = wz[hw - 1 - m], zr = wz[hw + m];
                        const float xl = frac + (float)m, xr = x1 - (float)m;
                        const float rl = sg * __builtin_amdgcn_rcpf(xl), rx = -sg * __builtin_amdgcn_rcpf(xr);
                        a1.x += rl * zl.x + rx * zr.x;
                        a1.y += rl * zl.y + rx * zr.y;
                        if (GRAD) {
                            // (-1)^m / x^2 = sg rl^2, and -sg rx^2 on the right
                            const float ql = sg * rl * rl, qr = -sg * rx * rx;
                            a2.x += ql * zl.x + qr * zr.x;
                            a2.y += ql * zl.y + qr * zr.y;
                            a0.x += sg * (zl.x - zr.x);
                            a0.y += sg * (zl.y - zr.y);
                            if constexpr (BIN) {
                                ax.x += sg * (xl * zl.x - xr * zr.x);
                                ax.y += sg * (xl * zl.y - xr * zr.y);
                            }
                        }
                    };
                    int m = 1;
                    for (; m + 1 < hw; m += 2) {
                        pair(m, -1.f);
                        pair(m + 1, 1.f);
                    }
                    if (m < hw) pair(m, -1.f);
                    const float sp = sf * (1.f / kPiF);
                    zt = make_float2(sp * a1.x + (w0_ * za.x + w1_ * zb.x), sp * a1.y + (w0_ * za.y + w1_ * zb.y));
                    if (GRAD) {
                        s1 = make_float2(cf * a1.x - sp * a2.x + (dw0 * za.x + dw1 * zb.x),
                                         cf * a1.y - sp * a2.y + (dw0 * za.y + dw1 * zb.y));
                        // w (p - u) = -w x = -(-1)^m sin(pi f) / pi
                        m1 = make_float2(-sp * (a0.x + za.x - zb.x), -sp * (a0.y + za.y - zb.y));
                        if constexpr (BIN)
                            m2 = make_float2(sp * (ax.x + frac * za.x - x1 * zb.x), sp * (ax.y + frac * za.y - x1 * zb.y));
                    }
                } else {
                    zt = make_float2(0.f, 0.f);
                    for (int i = 1; i <= W; ++i) {
                        const float x = frac + (float)(hw - i);
                        const bool odd = (hw - i) & 1;
                        const float sx = odd ? -sf : sf, cx = odd ? -cf : cf;  // sin, cos of pi x
                        float w, dw = 0.f;
                        if (x == 0.f) {
                            w = 1.f;
                        } else if (dir_series) {
                            // Dirichlet kernel of a long series: sinc(x) g(y), y = pi x / n
                            // small, g = y / tan(y) (n even) or y / sin(y) (n odd) as a series
                            float s0, ds0;
                            sinc_d(x, sx, cx, s0, ds0);
                            const float y = x * pin, y2 = y * y;
                            const float g = A.ip.n_odd ? 1.f + y2 * (1.f / 6.f + y2 * (7.f / 360.f))
                                                       : 1.f - y2 * (1.f / 3.f + y2 * (1.f / 45.f));
                            w = s0 * g;
                            if (GRAD) {
                                const float dg = A.ip.n_odd ? y * (1.f / 3.f + y2 * (7.f / 90.f))
                                                            : -y * (2.f / 3.f + y2 * (4.f / 45.f));
                                dw = ds0 * g + s0 * dg * pin;
                            }
                        } else {
                            kernel_w<GRAD>(A.ip, x, sx, cx, w, dw);
                        }
                        const float2 zz = wz[i - 1];
                        zt.x += w * zz.x;
                        zt.y += w * zz.y;
                        if (GRAD) {
                            s1.x += dw * zz.x;
                            s1.y += dw * zz.y;
                            const float wx = w * x;
                            m1.x -= wx * zz.x;
                            m1.y -= wx * zz.y;
                            if constexpr (BIN) {
                                m2.x += wx * x * zz.x;
                                m2.y += wx * x * zz.y;
                            }
                        }
                    }
                }
                bool mk = v.gap != 1;
                {
                    const double fn = floor(u + 0.5);
                    mk = mk && fn >= 0.0 && fn < (double)A.n;
                    if (v.gap == 2) mk = mk && !in_gap(A.gaps[X], A.n_gaps[X], (int64_t)fn);
                }
                // total phase: spindown Phi_s and the Fourier kernel at f;
                // us[j] = T^(j+2)/(j+2)! + d T^(j+1)/(j+1)! (cycles per unit f^(j+1))
                const double tb = (double)k * A.dt, d = V * A.dt, T = tb - d;
                double us[ORDER];
                double cyc = (f - A.f_het) * tb;
                if constexpr (ORDER == 1) {
                    us[0] = 0.5 * (tb * tb - d * d);
                    cyc += fs[0] * us[0];
                } else {
                    double Tj = T;  // T^(j+1)
#pragma unroll
                    for (int i = 0; i < ORDER; ++i) {
                        us[i] = Tj * T * kInvFact[i + 2] + d * Tj * kInvFact[i + 1];
                        cyc += fs[i] * us[i];
                        Tj *= T;
                    }
                }
                const float ph = (float)(cyc - rint(cyc));
                const float sn = __builtin_amdgcn_sinf(ph), cs = __builtin_amdgcn_cosf(ph);  // revolutions
                // times exp(-2 pi i cyc)
                auto turn = [&](float2 z, double& re, double& im) {
                    re = (double)(z.x * cs + z.y * sn);
                    im = (double)(z.y * cs - z.x * sn);
                };
                double zr, zi;
                turn(zt, zr, zi);
                const double av = quartic(v.poly[1], s), bv = quartic(v.poly[2], s);
                const double wa = D.w * av, wb = D.w * bv;
                acc[S_FA + 0] += wa * zr;
                acc[S_FA + 1] += wa * zi;
                acc[S_FB + 0] += wb * zr;
                acc[S_FB + 1] += wb * zi;
                if (mk) {
                    acc[S_A] += wa * av;
                    acc[S_B] += wb * bv;
                    acc[S_C] += wa * bv;
                }
                if constexpr (GRAD) {
                    // d/df: -2 pi i t_b, d/df^(j): -2 pi i us[j-1]; (-i c)(x + i y) = c y - i c x
                    auto phase_slope = [&](int i, double c) {
                        const double x = c * zi, y = -c * zr;
                        acc[S_DFA + 2 * i] += wa * x;
                        acc[S_DFA + 2 * i + 1] += wa * y;
                        acc[S_DFB + 2 * i] += wb * x;
                        acc[S_DFB + 2 * i + 1] += wb * y;
                    };
                    phase_slope(0, 2.0 * kPi * tb);
                    // dPhi_s/dT / (2 pi d) = sum_j f^(j) T^(j-1)/(j-1)!
                    double rate = 0.0, Tj = 1.0;
#pragma unroll
                    for (int i = 0; i < ORDER; ++i) {
                        phase_slope(1 + i, 2.0 * kPi * us[i]);
                        rate += fs[i] * Tj * kInvFact[i];
                        Tj *= T;
                    }
                    double sr, si, mr, mi, nr = 0.0, ni = 0.0;
                    turn(s1, sr, si);
                    turn(m1, mr, mi);
                    if constexpr (BIN) turn(m2, nr, ni);
                    // everything proportional to dT: s1 / dt - i H z~, with
                    // H = -2 pi f_het G + 2 pi rate d
                    double G = v.G[0] + s * v.G[1];
                    if constexpr (BIN) G += s * s * v.G[2];
                    const double H = 2.0 * kPi * (rate * d - A.f_het * G), inv_dt = A.inv_dt;
                    const double Qr = sr * inv_dt + H * zi, Qi = si * inv_dt - H * zr;
#pragma unroll
                    for (int i = 0; i < NS; ++i) {
                        const double dT = quartic(v.poly[3 + i], s);
                        const double da = D.w * quartic(v.poly[3 + NS + i], s);
                        const double db = D.w * quartic(v.poly[3 + 2 * NS + i], s);
                        double psi = v.psi[i][0];
                        if constexpr (BIN) psi += s * v.psi[i][1];
                        double Pr = dT * Qr + psi * mi, Pi = dT * Qi - psi * mr;
                        if constexpr (BIN) {
                            Pr += v.psi[i][2] * ni;
                            Pi -= v.psi[i][2] * nr;
                        }
                        acc[S_DFA + S_SKY + 2 * i] += da * zr + wa * Pr;
                        acc[S_DFA + S_SKY + 2 * i + 1] += da * zi + wa * Pi;
                        acc[S_DFB + S_SKY + 2 * i] += db * zr + wb * Pr;
                        acc[S_DFB + S_SKY + 2 * i + 1] += db * zi + wb * Pi;
                        if (mk) {
                            acc[S_DA + i] += 2.0 * da * av;
                            acc[S_DB + i] += 2.0 * db * bv;
                            acc[S_DC + i] += da * bv + db * av;
                        }
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();  // the next run rewrites this wave's window
        }
    }
    if (__any(overflow) && lane == 0) atomicOr(A.flags, 2u);

    // workgroup sums in a fixed order
    const double t = wave_sums<LOG2>(acc, lane);
    const int slot = lane >> (6 - LOG2);
    if ((lane & ((1 << (6 - LOG2)) - 1)) == 0 && slot < NSUM) red[wave][slot] = t;
    __syncthreads();
    if (tid < NSUM)
        A.partials[((int64_t)cand * A.n_blocks + blockIdx.x) * kPointSums + tid] =
            ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
}

// One workgroup per candidate: fixed-order sum of the block partials, then
// 2F = 2Q/D with Q = B|Fa|^2 + A|Fb|^2 - 2C Re(Fa Fb^*), D = AB - C^2, and
// d2F = 2 (dQ D - Q dD) / D^2.
// Thread (group, slot): a group's threads read whole rows of partial sums, the
// 16 groups stride over the rows, and their sums are added in a fixed order
// (one slot after another with a tree of 256 threads each took 15 to 26 us).
template <int ORDER, bool BIN>
__global__ __launch_bounds__(1024) void rsf_point_reduce_k(PointReduceArgs R) {
    using SL = Slots<ORDER, BIN>;
    constexpr int NP = SL::NP;
    constexpr int S_FA = SL::FA, S_FB = SL::FB, S_A = SL::A, S_B = SL::B, S_C = SL::C;
    constexpr int S_DFA = SL::DFA, S_DFB = SL::DFB, S_DA = SL::DA, S_DB = SL::DB, S_DC = SL::DC;
    constexpr int kGroups = 1024 / kPointSums;
    __shared__ double part[kGroups][kPointSums];
    __shared__ double tot[kPointSums];
    const int cand = blockIdx.x;
    const int nsum = R.grad ? SL::USED : S_DFA;
    const int slot = threadIdx.x % kPointSums, group = threadIdx.x / kPointSums;
    const double* p = R.partials + (int64_t)cand * R.n_blocks * kPointSums;
    {
        double v = 0.0;
        if (slot < nsum)
            for (int b = group; b < R.n_blocks; b += kGroups) v += p[(int64_t)b * kPointSums + slot];
        part[group][slot] = v;
    }
    __syncthreads();
    if (threadIdx.x < kPointSums) {
        double v = 0.0;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) v += part[g][threadIdx.x];
        tot[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double Far = tot[S_FA], Fai = tot[S_FA + 1], Fbr = tot[S_FB], Fbi = tot[S_FB + 1];
    const double Aa = tot[S_A], Bb = tot[S_B], Cc = tot[S_C];
    const double D = Aa * Bb - Cc * Cc;
    const double fa2 = Far * Far + Fai * Fai, fb2 = Fbr * Fbr + Fbi * Fbi;
    const double reab = Far * Fbr + Fai * Fbi;
    const double Q = Bb * fa2 + Aa * fb2 - 2.0 * Cc * reab;
    const bool degenerate = !(D > 0.0);
    const double F2 = degenerate ? __longlong_as_double(0x7ff8000000000000LL) : 2.0 * Q / D;
    if (degenerate) atomicOr(R.flags, 1u);
    if (R.twoF) R.twoF[cand] = (float)F2;
    if (!R.grad) return;
    const double g = (double)R.g_twoF[cand];
    for (int i = 0; i < NP; ++i) {
        const double dar = tot[S_DFA + 2 * i], dai = tot[S_DFA + 2 * i + 1];
        const double dbr = tot[S_DFB + 2 * i], dbi = tot[S_DFB + 2 * i + 1];
        // the antenna sums depend only on the parameters that move T (the last NS)
        const int k = i - (NP - SL::NS);
        const double dA = (k >= 0) ? tot[S_DA + k] : 0.0;
        const double dB = (k >= 0) ? tot[S_DB + k] : 0.0;
        const double dC = (k >= 0) ? tot[S_DC + k] : 0.0;
        const double dQ = dB * fa2 + 2.0 * Bb * (Far * dar + Fai * dai) + dA * fb2 +
                          2.0 * Aa * (Fbr * dbr + Fbi * dbi) - 2.0 * dC * reab -
                          2.0 * Cc * (dar * Fbr + dai * Fbi + Far * dbr + Fai * dbi);
        const double dD = dA * Bb + Aa * dB - 2.0 * Cc * dC;
        const double d2F = degenerate ? F2 : 2.0 * (dQ * D - Q * dD) / (D * D);
        R.g_theta[(int64_t)NP * cand + i] = g * d2F;
    }
}

// Rows of 64 samples per wave: whole runs of four rows, eight runs for long
// series (the node chain and the sums of a workgroup are shared by 128 rows)
// down to one, so that a candidate alone has around 128 to 256 workgroups; very
// short series put one row on each wave (n = 21,600: 85 workgroups instead of
// 22).  A candidate's split depends on the series alone: its result does not
// change with the number of candidates in a call.
int point_rows(int64_t P) { return P <= 512 ? 1 : P <= 4096 ? 4 : P <= 8192 ? 8 : P <= 16384 ? 16 : 32; }
int point_blocks(int64_t P, int rows) { return (int)((P + 4 * rows - 1) / (4 * rows)); }

// sampling intervals up to 4.4 s
bool point_interpolates(double dt, const EphDev& e) { return chain_interpolates(e, PointRun::half * dt, kDelayErr, 4e-9); }

hipError_t launch_point(const PointArgs& a, bool grad, hipStream_t s) {
    const dim3 grid((unsigned)a.n_blocks, (unsigned)a.n_cand);
#define RSF_POINT(K, G, O, B) hipLaunchKernelGGL((K<G, O, B>), grid, dim3(kThreads), 0, s, a)
#define RSF_POINT_CASES(K)                              \
    switch (a.order * 4 + (a.binary ? 2 : 0) + (grad ? 1 : 0)) { \
        case 4: RSF_POINT(K, false, 1, false); break;   \
        case 5: RSF_POINT(K, true, 1, false); break;    \
        case 6: RSF_POINT(K, false, 1, true); break;    \
        case 7: RSF_POINT(K, true, 1, true); break;     \
        case 8: RSF_POINT(K, false, 2, false); break;   \
        case 9: RSF_POINT(K, true, 2, false); break;    \
        case 10: RSF_POINT(K, false, 2, true); break;   \
        case 11: RSF_POINT(K, true, 2, true); break;    \
        case 12: RSF_POINT(K, false, 3, false); break;  \
        case 13: RSF_POINT(K, true, 3, false); break;   \
        case 14: RSF_POINT(K, false, 3, true); break;   \
        case 15: RSF_POINT(K, true, 3, true); break;    \
        default: return hipErrorInvalidValue;           \
    }
    if (a.run) {
        RSF_POINT_CASES(rsf_point_run_k)
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || !a.binary) return e;
    }
    // a binary plan's candidates choose their kernel on the device, by their orbit
    RSF_POINT_CASES(rsf_point_k)
#undef RSF_POINT_CASES
#undef RSF_POINT
    return hipGetLastError();
}

hipError_t launch_point_reduce(const PointReduceArgs& r, hipStream_t s) {
    const dim3 grid((unsigned)r.n_cand);
#define RSF_POINT_REDUCE(O, B) hipLaunchKernelGGL((rsf_point_reduce_k<O, B>), grid, dim3(1024), 0, s, r)
    switch (r.order * 2 + (r.binary ? 1 : 0)) {
        case 2: RSF_POINT_REDUCE(1, false); break;
        case 3: RSF_POINT_REDUCE(1, true); break;
        case 4: RSF_POINT_REDUCE(2, false); break;
        case 5: RSF_POINT_REDUCE(2, true); break;
        case 6: RSF_POINT_REDUCE(3, false); break;
        case 7: RSF_POINT_REDUCE(3, true); break;
        default: return hipErrorInvalidValue;
    }
#undef RSF_POINT_REDUCE
    return hipGetLastError();
}

}  // namespace rsf
