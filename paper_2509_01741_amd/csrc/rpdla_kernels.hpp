// rpdla_kernels.hpp -- HIP kernels for gfx950 (wave64): atom sampling,
// ionization times, the Newton-Lorentz push (double and mixed precision) and
// the energy-angle histogram.
#pragma once

#include <type_traits>

#include "rpdla_device.hpp"
#include "rpdla_plan.hpp"

namespace rpdla {

constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr double kInvTwoPi = 0.15915494309189533576888376337251;

// ---------------------------------------------------------------------------
// Atom sampling: one lane per atom, structure-of-arrays output.
// r = R sqrt(u0), azimuth 2 pi u1, z = zh (2 u2 - 1)  (Sec. 2.1).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) sample_atoms_kernel(
    uint64_t seed, uint32_t cfg, uint64_t first_atom, int64_t n, double r_max, double z_half,
    double* __restrict__ x, double* __restrict__ y, double* __restrict__ z)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const U64x4 r = philox4x64(first_atom + (uint64_t)i, 0, 0, 0, seed, (uint64_t)cfg);
    const double rad = r_max * sqrt(u01(r.v[0]));
    double sn, cs;
    sincos(kTwoPi * u01(r.v[1]), &sn, &cs);
    x[i] = rad * cs;
    y[i] = rad * sn;
    z[i] = z_half * (2.0 * u01(r.v[2]) - 1.0);
}

// Annulus: r uniform in area between r_in and r_out (r = r_out exactly when
// r_in == r_out, a hollow-cylinder surface), azimuth and z as above.
__global__ void __launch_bounds__(256) sample_annulus_kernel(
    uint64_t seed, uint32_t cfg, uint64_t first_atom, int64_t n, double r_in, double r_out,
    double z_half, double* __restrict__ x, double* __restrict__ y, double* __restrict__ z)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const U64x4 r = philox4x64(first_atom + (uint64_t)i, 0, 0, 0, seed, (uint64_t)cfg);
    const double rad = (r_in == r_out) ? r_out
                                        : sqrt(r_in * r_in + u01(r.v[0]) * (r_out * r_out - r_in * r_in));
    double sn, cs;
    sincos(kTwoPi * u01(r.v[1]), &sn, &cs);
    x[i] = rad * cs;
    y[i] = rad * sn;
    z[i] = z_half * (2.0 * u01(r.v[2]) - 1.0);
}

// Laser phase at each birth, the phase defined under Eq. (2) of the paper
// (k z - omega t - 2 atan(z/z_r) + z r^2/(z_r w0^2 f^2), with the paper's
// carrier phase equal to minus this library's), in [0, 2 pi), and the radius
// of the parent ion (optional); NaN for unborn slots.
__global__ void __launch_bounds__(256) birth_phase_kernel(
    DevCfg c, int64_t n, const double* __restrict__ tb, const double* __restrict__ x,
    const double* __restrict__ y, const double* __restrict__ z, int spa,
    double* __restrict__ phase, double* __restrict__ r_birth)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const double t = tb[s];
    const int64_t a = s / spa;
    const bool born = t < __builtin_inf();
    if (r_birth) r_birth[s] = born ? sqrt(x[a] * x[a] + y[a] * y[a]) : __builtin_nan("");
    if (!born) { phase[s] = __builtin_nan(""); return; }
    const double X = x[a] * c.k, Y = y[a] * c.k, Z = z[a] * c.k;
    const double rho2 = (X * X + Y * Y) * c.inv_w0n2;
    const double zeta = Z * c.inv_zrn;
    double ph = Z - t * c.omega - 2.0 * atan(zeta) + zeta * rho2 / (1.0 + zeta * zeta) - c.phi0;
    ph = fmod(ph, kTwoPi);
    if (ph < 0.0) ph += kTwoPi;
    if (ph >= kTwoPi) ph -= kTwoPi;
    phase[s] = ph;
}

// ---------------------------------------------------------------------------
// Ionization.  One wave per atom.  Time axis in panels of width h from the
// window start; state s (charge state k_first + s) accumulates GL-4 panel
// integrals of its rate from the previous birth; at the panel where the sum
// reaches the Exp(1) threshold the crossing is solved by bracketed Newton.
// Panels where a rigorous bound keeps the rate negligible at every node are
// skipped: before each state's possible window and after it.
// ---------------------------------------------------------------------------
template <int FIELD, class CFG>
__device__ inline double emag2_f64(const CFG& c, double X, double Y, double Z, double d)
{
    double ax, ay, az, bx, by, bz;
    field_f64<FIELD, false, CFG>(c, X, Y, Z, d, ax, ay, az, bx, by, bz);
    return ax * ax + ay * ay + az * az;
}

// The field of an atom at rest reduced to its time dependence.  For the RP
// models every term of the series is g e^{i Psi} q^n times a polynomial in
// rho^2, so  Er/r ~ g Re(e^{i Psi} A_E),  Ez = g Im(e^{i Psi} A_Z)  with the
// complex position factors A_E = q^2 P_E(q), A_Z = q^2 P_Z(q) (the push's
// series coefficients regrouped by powers of q), g = a0 exp(-rho^2/D - s^2)
// and Psi = tau + psi_c: one sine/cosine and one exponential per time.
struct AtomGeom {
    double X, Y, Z;
    double r2, mrD, psi_c;
    double aer, aei, azr, azi;
};

template <int FIELD, class CFG>
__device__ inline AtomGeom atom_geom(const CFG& c, double X, double Y, double Z)
{
    AtomGeom a{X, Y, Z, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if constexpr (FIELD == 1 || FIELD == 3 || FIELD == 5) {
        const double r2 = (X * X + Y * Y) * c.inv_w0n2;
        const double zeta = Z * c.inv_zrn;
        const double iD = 1.0 / (1.0 + zeta * zeta);
        const double rD = r2 * iD;
        a.r2 = r2;
        a.mrD = -rD;
        a.psi_c = c.phi0 - rD * zeta;
        const Cx<double> q{iD, zeta * iD};
        const double r4 = r2 * r2, r6 = r4 * r2, r8 = r4 * r4;
        // P_E(q) = sum p_n q^n and P_Z(q) = sum z_n q^n, by Horner in q
        // Horner step: p <- p q + coefficient
        auto horner = [&q](Cx<double> p, double coef) {
            const Cx<double> t = cmul(p, q);
            return Cx<double>{t.re + coef, t.im};
        };
        Cx<double> pe{1.0, 0.0}, pz{c.eps, 0.0};
        if constexpr (FIELD == 1) {
            pz = horner(Cx<double>{-c.eps * r2, 0.0}, c.eps);
        } else {
            double p[7] = {1.0, -0.5 * c.e2, c.e2 * r2, -0.25 * c.e2 * r4, 0.0, 0.0, 0.0};
            if constexpr (FIELD == 5) {
                p[2] += -0.375 * c.e4;
                p[3] += -0.375 * c.e4 * r2;
                p[4] = 1.0625 * c.e4 * r4;
                p[5] = -0.375 * c.e4 * r6;
                p[6] = 0.03125 * c.e4 * r8;
            }
            const double z[5] = {c.eps, -c.eps * r2 + 0.5 * c.e3, 0.5 * c.e3 * r2,
                                 -1.25 * c.e3 * r4, 0.25 * c.e3 * r6};
            constexpr int NE = (FIELD == 5) ? 7 : 4;
            pe = Cx<double>{p[NE - 1], 0.0};
#pragma unroll
            for (int n = NE - 2; n >= 0; --n) pe = horner(pe, p[n]);
            pz = Cx<double>{z[4], 0.0};
#pragma unroll
            for (int n = 3; n >= 0; --n) pz = horner(pz, z[n]);
        }
        const Cx<double> q2 = cmul(q, q);
        const Cx<double> ae = cmul(q2, pe), az = cmul(q2, pz);
        a.aer = ae.re; a.aei = ae.im; a.azr = az.re; a.azi = az.im;
    }
    return a;
}

template <int FIELD, class CFG, class RCFG>
__device__ inline double emag2_atom(const CFG& c, const RCFG& rc, const AtomGeom& a, double d,
                                    const fm::Coef& k = fm::kCoef)
{
    if constexpr (FIELD == 1 || FIELD == 3 || FIELD == 5) {
        const double s = d * rc.inv_T0n;
        const double g = rc.a0 * fm::exp_fin_f64(a.mrD - s * s, k);
        // the sign (-1)^n of the half-angle form cancels in the squares
        double sg, kp;
        fm::cis_half2_f64(d, a.psi_c, &sg, &kp, k);
        const double cs = fma(-sg, sg, 1.0), sn = sg * kp;
        // one product of each sum fused, as stated: birth times then do not
        // depend on how the kernel around this is compiled
        const double et = rc.er_scale * g * fma(a.aer, cs, -(a.aei * sn));
        const double ez = rc.ez_scale * g * fma(a.azr, sn, a.azi * cs);
        return fma(ez, ez, et * et * a.r2);
    } else {
        return emag2_f64<FIELD>(c, a.X, a.Y, a.Z, d);
    }
}

// Panel range [j_lo, j_hi] outside which the state's ln w lies below the skip
// level (adk_a2thr) at every node.
template <class CFG>
RPDLA_HD inline bool state_window(const CFG& c, const AdkState& st, double bound2, double Zc,
                                    double tau_s, double h, int32_t M, int32_t& j_lo, int32_t& j_hi)
{
    const double thr = st.a2thr;
    if (!(bound2 >= thr)) return false;            // never reaches a nonzero rate
    if (c.field == 11) { j_lo = 0; j_hi = M - 1; return true; }
    const double smax = sqrt(0.5 * log(bound2 / thr));
    const double half = smax / c.inv_T0n;          // in normalized time
    const double lo = floor((Zc - half - tau_s) / h) - 1.0;
    const double hi = ceil((Zc + half - tau_s) / h) + 1.0;
    j_lo = lo < 0.0 ? 0 : (lo > (double)(M - 1) ? M - 1 : (int32_t)lo);
    j_hi = hi > (double)(M - 1) ? M - 1 : (hi < 0.0 ? 0 : (int32_t)hi);
    return true;
}

// Upper bound of what the panel loop below can add up for state st over the
// panels j0..j1 (the first one from d_from): a panel's GL-4 estimate is at
// most its width times the largest rate at its nodes, and the rate is at
// most the ADK rate at the largest |a|^2 the field bound allows there,
// |a|^2 <= b2 exp(-2 s^2) (lb2 = ln b2), capped at the |a|^2 where the rate
// itself peaks.  Panels go in groups of kBoundGroup (one optical period);
// each group is charged its width times that rate at its smallest |s|.  When
// twice this bound stays below the state's threshold the loop could not reach
// it: the state, and so every later one, is never born, which is what
// integrating all the panels would give.  never_reaches() answers that.  It
// takes the group nearest the envelope peak (s = 0) first, the largest term,
// and stops as soon as the sum passes half the threshold, so a state that
// will be born costs one or two groups.
constexpr int32_t kBoundGroup = 200;

// Edges of group g (0-based) of panels j0..j1, as the panel loop forms its
// panel edges: from d_from or panel j0 + g kBoundGroup to the start of the
// next group or the end of panel j1.
RPDLA_HD inline void bound_group(int32_t g, int32_t groups, int32_t j0, int32_t j1, int32_t M,
                                   double d_s, double d_e, double h, double d_from, double& da,
                                   double& db)
{
    da = (g == 0) ? d_from : d_s + (double)(j0 + g * kBoundGroup) * h;
    db = (g + 1 < groups) ? d_s + (double)(j0 + (g + 1) * kBoundGroup) * h
                          : ((j1 == M - 1) ? d_e : d_s + (double)(j1 + 1) * h);
}

template <class CFG>
RPDLA_HD inline double bound_group_rate(const CFG& c, const AdkState& st, double lb2, double la2pk,
                                          double da, double db)
{
    const double smin = (da <= 0.0 && db >= 0.0) ? 0.0 : fmin(fabs(da), fabs(db)) * c.inv_T0n;
    const double la2 = fmin(lb2 - 2.0 * smin * smin, la2pk);
    const double lw = st.c0 - st.c1h * la2 - st.c2 * fm::exp_f64(-0.5 * la2);
    return (db - da) * fm::exp_f64(lw);
}

template <class CFG>
__device__ inline bool never_reaches(const CFG& c, const AdkState& st, double lb2, double d_s,
                                     double d_e, double h, int32_t M, int32_t j0, int32_t j1,
                                     double d_from, double target)
{
    // ln |a|^2 where ln w = c0 - c1h ln|a|^2 - c2 |a|^-1 peaks
    const double la2pk = (st.c1h > 0.0) ? 2.0 * fm::log_pos_f64(st.c2 / (2.0 * st.c1h))
                                         : __builtin_inf();
    const int32_t groups = (j1 - j0) / kBoundGroup + 1;
    // the group holding d = 0, or the one nearest to it
    const double jpk = floor(-d_s / h) - (double)j0;
    const int32_t gpk = jpk <= 0.0 ? 0
                      : (jpk >= (double)(groups - 1) * kBoundGroup ? groups - 1
                                                                   : (int32_t)jpk / kBoundGroup);
    double da, db;
    bound_group(gpk, groups, j0, j1, M, d_s, d_e, h, d_from, da, db);
    double sum = bound_group_rate(c, st, lb2, la2pk, da, db);
    if (!(2.0 * sum < target)) return false;
#pragma unroll 1
    for (int32_t g = 0; g < groups; ++g) {
        if (g == gpk) continue;
        bound_group(g, groups, j0, j1, M, d_s, d_e, h, d_from, da, db);
        sum += bound_group_rate(c, st, lb2, la2pk, da, db);
        if (!(2.0 * sum < target)) return false;
    }
    return true;
}

// v of one lane (uniform index), the same in every lane.
__device__ inline double lane_value(double v, int lane)
{
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// I <- fma(h_l, acc_l, I) for l = 0..15 of each row of 16 lanes in turn (h_l,
// acc_l the values of the row's lane l), in every lane of the row.  Two
// instructions a term: a 64-bit row broadcast of h_l, and the multiply-add
// that broadcasts acc_l as it reads it.
#if defined(__HIP_DEVICE_COMPILE__)
#define RPDLA_ROW_TERM(L)                                                                      \
    "v_mov_b64_dpp %1, %2 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"                 \
    "v_fmac_f64_dpp %0, %3, %1 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
__device__ inline double row_sum(double I, double h, double acc)
{
    double t;
    // two wait states between the write of a register and its read by another lane
    asm("s_nop 1\n\t" RPDLA_ROW_TERM(0) RPDLA_ROW_TERM(1) RPDLA_ROW_TERM(2) RPDLA_ROW_TERM(3)
        RPDLA_ROW_TERM(4) RPDLA_ROW_TERM(5) RPDLA_ROW_TERM(6) RPDLA_ROW_TERM(7)
        RPDLA_ROW_TERM(8) RPDLA_ROW_TERM(9) RPDLA_ROW_TERM(10) RPDLA_ROW_TERM(11)
        RPDLA_ROW_TERM(12) RPDLA_ROW_TERM(13) RPDLA_ROW_TERM(14) RPDLA_ROW_TERM(15)
        : "+v"(I), "=&v"(t) : "v"(h), "v"(acc));
    return I;
}
#undef RPDLA_ROW_TERM
#else
__device__ double row_sum(double I, double h, double acc);
#endif

// Constants of the rate evaluation: the configuration's, and those of the
// functions, which stay in registers as in StepRegs (49 doubles; with the
// compiler's own choice a node took 160 vector instructions, 22 of them moves
// of coefficients, and its scalar loads; now 131, at 3 waves per SIMD).
struct RateRegs {
    double inv_T0n, a0, er_scale, ez_scale, gl_x[2], gl_w[2], lnw_zero;
    fm::Coef k;
    fm::LogCoef l;
    template <class CFG>
    __device__ inline explicit RateRegs(const CFG& c)   // nodes and weights are symmetric
        : inv_T0n(c.inv_T0n), a0(c.a0), er_scale(c.er_scale), ez_scale(c.ez_scale),
          gl_x{c.gl_x[2], c.gl_x[3]}, gl_w{c.gl_w[2], c.gl_w[3]}, lnw_zero(c.lnw_zero)
    {
        keep_in_vgpr(k.magic);
        keep_in_sgpr(k.log2e); keep_in_sgpr(k.nln2_1); keep_in_sgpr(k.nln2_2);
#pragma unroll
        for (int i = 0; i < 10; ++i) if (i == 8) keep_in_vgpr(k.ex[i]); else keep_in_sgpr(k.ex[i]);
        keep_in_sgpr(k.inv_pi); keep_in_sgpr(k.npi_1); keep_in_sgpr(k.npi_2);
        keep_in_vgpr(k.npi_3);
#pragma unroll
        for (int i = 0; i < 7; ++i) keep_in_vgpr(k.sg[i]);
#pragma unroll
        for (int i = 0; i < 6; ++i) if (i >= 4) keep_in_vgpr(k.kp[i]); else keep_in_sgpr(k.kp[i]);
        keep_in_vgpr(k.ns2o8); keep_in_vgpr(k.s2);
        keep_in_vgpr(k.c375);
        keep_in_vgpr(l.rsqrt2);
#pragma unroll
        for (int i = 0; i < 9; ++i) keep_in_vgpr(l.at[i]);
    }
};

// Birth times of one atom (index `atom`, normalized position X, Y, Z) for
// states k_first..k_first+K-1, written to out[0..K) in seconds; called by a
// whole wave.  The atom is at rest, so its field depends on time only through
// the retarded time d = tau - Z: the panels, nodes and crossings are all taken
// in d (the same grid as in tau, shifted by Z), so the carrier phase is formed
// from d itself and the birth time tau = d + Z is rounded once, at the output.
//
// The lanes take 64 consecutive panels of one state at a time and the panel
// integrals are added up in the panels' order, so the sums are those of one
// lane that takes panel after panel.  An atom has a few thousand panels and
// about nine births (bound: FP64 issue; four nodes of 131 instructions a
// panel, one in fourteen evaluated past a crossing; 200 of the 750
// instructions for 64 panels go into the ordered sum).  With one lane per atom
// a wave's lanes waited for one another (37 of 64 at work) and a small
// ensemble left most of the chip idle behind one lane's serial chain: 1024
// atoms x 8 states 11.7 -> 0.13 ms, 2e5 atoms x 1 state 11.8 -> 7.6 ms, 1e6
// atoms x 10 states 147 -> 119 ms.  ionize_form says where the forms below take
// its place.
template <int FIELD, class CFG>
__device__ void ionize_atom(const CFG& c, const RateRegs& R, uint64_t seed, uint32_t cfg,
                                 uint64_t atom, double X, double Y, double Z, int k_first, int K,
                                 double* __restrict__ out)
{
    const int lane = __lane_id();
    // lane s holds what belongs to state s: threshold, constants, panel window
    // and whether its rate bound leaves it open from the window start
    const double dz = (c.window == 0) ? 0.0 : -Z;
    const double d_s = dz - c.tb_n, d_e = dz + c.ta_n;
    const double h = c.hn;
    const int32_t M = (int32_t)ceil((d_e - d_s) / h);
    const double b2 = bound2_f64<FIELD>(c, X, Y, Z);
    const double lb2 = fm::log_pos_f64(b2);
    double tbirth = __builtin_inf(), tgt_l = 0.0;
    AdkState st_l{0.0, 0.0, 0.0, 0.0, 0.0};
    int32_t jlo_l = 0, jhi_l = 0;
    bool win_l = false, open_l = false;
    if (lane < K) {
        tgt_l = -log(uniform_j(seed, cfg, atom, k_first + lane + 2));
        st_l = adk_state(c, k_first - 1 + lane);
        win_l = state_window(c, st_l, b2, 0.0, d_s, h, M, jlo_l, jhi_l);
        open_l = win_l && (FIELD == 11 || !never_reaches(c, st_l, lb2, d_s, d_e, h, M, jlo_l, jhi_l,
                                                         d_s + (double)jlo_l * h, tgt_l));
    }
    const uint64_t open = __ballot(open_l), late = __ballot(tgt_l > 0.0);

    int s = 0;
    while (s < K && !((late >> s) & 1)) {   // zero thresholds: born where they start
        if (lane == s) tbirth = (d_s + Z) * c.inv_omega;
        ++s;
    }
    if (s < K && ((open >> s) & 1)) {
        const AtomGeom ag = atom_geom<FIELD>(c, X, Y, Z);
        AdkState st{lane_value(st_l.c0, s), lane_value(st_l.c1h, s), lane_value(st_l.c2, s), 0.0,
                    R.lnw_zero};
        double target = lane_value(tgt_l, s);
        double I = 0.0, tstart = d_s;
        int32_t j = __builtin_amdgcn_readlane(jlo_l, s), j_hi = __builtin_amdgcn_readlane(jhi_l, s);
        auto rate = [&](double d) {
            return adk_rate_n(st, emag2_atom<FIELD>(c, R, ag, d, R.k), R.k, R.l);
        };
        while (j <= j_hi) {
            // lane: panel j + lane, its Gauss sum over [lo, b]
            const int32_t jl = j + lane;
            const double a = fma((double)jl, h, d_s);
            const double b = (jl == M - 1) ? d_e : fma((double)(jl + 1), h, d_s);
            const double lo = (tstart > a) ? tstart : a;
            const double hw = 0.5 * (b - lo), m = 0.5 * (lo + b);
            double acc = 0.0;
            if (jl <= j_hi) {
                acc = fma(R.gl_w[1], rate(fma(-R.gl_x[1], hw, m)), acc);
                acc = fma(R.gl_w[0], rate(fma(-R.gl_x[0], hw, m)), acc);
                acc = fma(R.gl_w[0], rate(fma(R.gl_x[0], hw, m)), acc);
                acc = fma(R.gl_w[1], rate(fma(R.gl_x[1], hw, m)), acc);
            }
            // add them up in order, row by row of 16 lanes; a row whose every
            // term is below a quarter of I's last place leaves I as it is
            const uint64_t counts = __ballot(!(hw * acc <= I * 0x1.0p-56));
            int cross = -1;
#pragma unroll 1
            for (int r = 0; r < 4; ++r) {
                if (((counts >> (16 * r)) & 0xffffull) == 0) continue;
                const double In = lane_value(row_sum(I, hw, acc), 16 * r);
                if (In < target) { I = In; continue; }
                // the crossing lies in this row: panel by panel
#pragma unroll 1
                for (cross = 16 * r; cross < 16 * r + 15; ++cross) {
                    const double Ix = fma(lane_value(hw, cross), lane_value(acc, cross), I);
                    if (!(Ix < target)) break;
                    I = Ix;
                }
                break;
            }
            if (cross < 0) { j += 64; continue; }
            // Newton for the crossing, bracketed, halving where a step leaves the
            // bracket: lanes 0..3 evaluate the Gauss nodes of [lo, t], lane 4 the
            // rate at t
            const double clo = lane_value(lo, cross), chi = lane_value(b, cross);
            const double chw = lane_value(hw, cross), cacc = lane_value(acc, cross);
            const double need = target - I;
            double t = clo;
            if (need > 0.0) {
                double tl = clo, th = chi;
                t = fma(chi - clo, need / (chw * cacc), clo);
                if (!(t > tl && t < th)) t = 0.5 * (tl + th);
                const double xn = (lane == 0) ? -R.gl_x[1] : (lane == 1) ? -R.gl_x[0]
                                : (lane == 2) ? R.gl_x[0] : R.gl_x[1];
#pragma unroll 1
                for (int it = 0; it < 100; ++it) {
                    const double hh = 0.5 * (t - clo), mm = 0.5 * (clo + t);
                    const double r = rate(lane < 4 ? fma(xn, hh, mm) : t);
                    double g = fma(R.gl_w[1], lane_value(r, 0), 0.0);
                    g = fma(R.gl_w[0], lane_value(r, 1), g);
                    g = fma(R.gl_w[0], lane_value(r, 2), g);
                    g = fma(R.gl_w[1], lane_value(r, 3), g);
                    const double gd = fma(hh, g, -need);
                    if (gd == 0.0) break;
                    if (gd > 0.0) th = t; else tl = t;
                    const double tol = ldexp(fmax(fabs(t), kTwoPi), -40);
                    const double w = lane_value(r, 4);
                    double tn = __builtin_nan("");
                    if (w > 0.0) {
                        const double dlt = gd / w;
                        if (fabs(dlt) <= tol) { t = t - dlt; break; }
                        tn = t - dlt;
                    }
                    if (!(tn > tl && tn < th)) tn = 0.5 * (tl + th);
                    const double step = fabs(tn - t);
                    t = tn;
                    if (step <= tol) break;
                }
            }
            if (lane == s) tbirth = (t + Z) * c.inv_omega;
            j += cross;
            ++s;
            // states with a zero threshold are born where the previous one is
            while (s < K && !((late >> s) & 1)) {
                if (lane == s) tbirth = (t + Z) * c.inv_omega;
                ++s;
            }
            if (s >= K || !((open >> s) & 1)) break;
            st.c0 = lane_value(st_l.c0, s);
            st.c1h = lane_value(st_l.c1h, s);
            st.c2 = lane_value(st_l.c2, s);
            target = lane_value(tgt_l, s);
            I = 0.0;
            tstart = t;
            const int32_t nlo = __builtin_amdgcn_readlane(jlo_l, s);
            j_hi = __builtin_amdgcn_readlane(jhi_l, s);
            const double d0 = nlo > j ? d_s + (double)nlo * h : t;
            if (nlo > j) j = nlo;
            if (FIELD != 11 && j <= j_hi) {
                // the rate bound over what is left of the window, a group of
                // panels per lane
                const double la2pk = (st.c1h > 0.0) ? 2.0 * fm::log_pos_f64(st.c2 / (2.0 * st.c1h))
                                                    : __builtin_inf();
                const int32_t groups = (j_hi - j) / kBoundGroup + 1;
                double sum = 0.0;
                for (int32_t g = lane; g < groups; g += 64) {
                    double da, db;
                    bound_group(g, groups, j, j_hi, M, d_s, d_e, h, d0, da, db);
                    sum += bound_group_rate(c, st, lb2, la2pk, da, db);
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
                if (2.0 * sum < target) break;
            }
        }
    }
    if (lane < K) out[lane] = tbirth;
}

template <int FIELD>
struct IonizeWaves { static constexpr int value = (FIELD > 20) ? 2 : 3; };

__device__ inline int64_t wave_index()
{
    return (int64_t)blockIdx.x * (blockDim.x >> 6) +
           __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

template <int FIELD>
__global__ void __launch_bounds__(256, IonizeWaves<FIELD>::value) ionize_kernel(
    DevCfg c, uint64_t seed, uint32_t cfg, uint64_t first_atom, int64_t n,
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    int k_first, int k_last, double* __restrict__ t_birth)
{
    const int64_t i = wave_index();
    if (i >= n) return;
    const int K = k_last - k_first + 1;
    const RateRegs R(c);
    ionize_atom<FIELD>(c, R, seed, cfg, first_atom + (uint64_t)i, x[i] * c.k, y[i] * c.k,
                       z[i] * c.k, k_first, K, t_birth + i * K);
}

// ---------------------------------------------------------------------------
// The other two forms of the ionization, for many atoms.  With a wave per atom
// the set-up of an atom (threshold, window, rate bound) costs a wave whatever
// comes of it, a birth throws away what was evaluated past it and its Newton
// iterations have five lanes at work; with hundreds of atoms for every SIMD the
// lanes have work of their own.  Each atom's arithmetic is the same in all forms.
// With only the wave form, ensembles that reach few states or have short windows
// took up to ten times what a lane per atom took before it (1e6 atoms at 7e14
// W/cm^2 4.2 ms instead of 0.34, with 2 fs pulses 32 instead of 26; now 0.09, 20).
// ---------------------------------------------------------------------------

// Birth times of one atom, as ionize_atom, by one lane: panel after panel.
template <int FIELD, class CFG>
__device__ void ionize_atom_lane(const CFG& c, const RateRegs& R, uint64_t seed, uint32_t cfg,
                                 uint64_t atom, double X, double Y, double Z, int k_first, int K,
                                 double* __restrict__ out)
{
    for (int s = 0; s < K; ++s) out[s] = __builtin_inf();
    const double dz = (c.window == 0) ? 0.0 : -Z;
    const double d_s = dz - c.tb_n, d_e = dz + c.ta_n;
    const double h = c.hn;
    const int32_t M = (int32_t)ceil((d_e - d_s) / h);
    const double b2 = bound2_f64<FIELD>(c, X, Y, Z);
    const double lb2 = fm::log_pos_f64(b2);
    auto threshold = [&](int s) { return -log(uniform_j(seed, cfg, atom, k_first + s + 2)); };
    int s = 0;
    double target = threshold(0);
    while (!(target > 0.0)) {               // zero thresholds: born where they start
        out[s] = (d_s + Z) * c.inv_omega;
        if (++s >= K) return;
        target = threshold(s);
    }
    AdkState st = adk_state(c, k_first - 1 + s);
    int32_t j, j_hi;
    if (!state_window(c, st, b2, 0.0, d_s, h, M, j, j_hi)) return;
    if (FIELD != 11 &&
        never_reaches(c, st, lb2, d_s, d_e, h, M, j, j_hi, d_s + (double)j * h, target))
        return;
    const AtomGeom ag = atom_geom<FIELD>(c, X, Y, Z);
    st.lnw_zero = R.lnw_zero;
    auto rate = [&](double d) {
        return adk_rate_n(st, emag2_atom<FIELD>(c, R, ag, d, R.k), R.k, R.l);
    };
    // Gauss sum over [m - hw, m + hw], in units of hw
    auto gauss = [&](double hw, double m) {
        double acc = 0.0;
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const bool outer = i == 0 || i == 3;
            const double x = outer ? R.gl_x[1] : R.gl_x[0];
            acc = fma(outer ? R.gl_w[1] : R.gl_w[0], rate(fma(i < 2 ? -x : x, hw, m)), acc);
        }
        return acc;
    };
    double I = 0.0, tstart = d_s;
    while (j <= j_hi) {
        const double a = fma((double)j, h, d_s);
        const double b = (j == M - 1) ? d_e : fma((double)(j + 1), h, d_s);
        const double lo = (tstart > a) ? tstart : a;
        const double hw = 0.5 * (b - lo);
        const double acc = gauss(hw, 0.5 * (lo + b));
        const double In = fma(hw, acc, I);
        if (In < target) {
            I = In;
            ++j;
            continue;
        }
        // bracketed Newton for the crossing, as in ionize_atom
        const double need = target - I;
        double t = lo;
        if (need > 0.0) {
            double tl = lo, th = b;
            t = fma(b - lo, need / (hw * acc), lo);
            if (!(t > tl && t < th)) t = 0.5 * (tl + th);
#pragma unroll 1
            for (int it = 0; it < 100; ++it) {
                const double hh = 0.5 * (t - lo);
                const double gd = fma(hh, gauss(hh, 0.5 * (lo + t)), -need);
                if (gd == 0.0) break;
                if (gd > 0.0) th = t; else tl = t;
                const double tol = ldexp(fmax(fabs(t), kTwoPi), -40);
                const double w = rate(t);
                double tn = __builtin_nan("");
                if (w > 0.0) {
                    const double dlt = gd / w;
                    if (fabs(dlt) <= tol) { t = t - dlt; break; }
                    tn = t - dlt;
                }
                if (!(tn > tl && tn < th)) tn = 0.5 * (tl + th);
                const double step = fabs(tn - t);
                t = tn;
                if (step <= tol) break;
            }
        }
        out[s] = (t + Z) * c.inv_omega;
        if (++s >= K) return;
        target = threshold(s);
        while (!(target > 0.0)) {
            out[s] = (t + Z) * c.inv_omega;
            if (++s >= K) return;
            target = threshold(s);
        }
        st = adk_state(c, k_first - 1 + s);
        st.lnw_zero = R.lnw_zero;
        I = 0.0;
        tstart = t;
        int32_t nlo;
        if (!state_window(c, st, b2, 0.0, d_s, h, M, nlo, j_hi)) return;
        const double d0 = nlo > j ? d_s + (double)nlo * h : t;
        if (nlo > j) j = nlo;
        if (FIELD != 11 && j <= j_hi &&
            never_reaches(c, st, lb2, d_s, d_e, h, M, j, j_hi, d0, target))
            return;
    }
}

// Whether the rate bound leaves any state of an atom open (ionize_atom would
// integrate, or write a birth at the window's start).
template <int FIELD, class CFG>
__device__ inline bool atom_open(const CFG& c, uint64_t seed, uint32_t cfg, uint64_t atom, double X,
                                 double Y, double Z, int k_first)
{
    const double dz = (c.window == 0) ? 0.0 : -Z;
    const double d_s = dz - c.tb_n, d_e = dz + c.ta_n;
    const int32_t M = (int32_t)ceil((d_e - d_s) / c.hn);
    const double b2 = bound2_f64<FIELD>(c, X, Y, Z);
    const double target = -log(uniform_j(seed, cfg, atom, k_first + 2));
    if (!(target > 0.0)) return true;
    const AdkState st = adk_state(c, k_first - 1);
    int32_t j_lo, j_hi;
    if (!state_window(c, st, b2, 0.0, d_s, c.hn, M, j_lo, j_hi)) return false;
    return FIELD == 11 || !never_reaches(c, st, fm::log_pos_f64(b2), d_s, d_e, c.hn, M, j_lo, j_hi,
                                         d_s + (double)j_lo * c.hn, target);
}

struct IonizeArgs {
    DevCfg c;
    uint64_t seed;
    uint32_t cfg;
    uint64_t first_atom;
    int64_t n;
    const double* x;
    const double* y;
    const double* z;
    int32_t k_first, K;
    double* out;
    int32_t per_wave;            // ionize_few_kernel: atoms of a wave, at most 64
    const uint32_t* order;       // ionize_lane_kernel
};

// Few atoms reach their first state: a wave asks the bound for per_wave atoms,
// one to a lane, and then takes those that it leaves open one after another.
template <int FIELD>
__global__ void __launch_bounds__(256, IonizeWaves<FIELD>::value) ionize_few_kernel(IonizeArgs A)
{
    const int lane = __lane_id();
    const int64_t i0 = wave_index() * A.per_wave;
    if (i0 >= A.n) return;
    const int64_t i = i0 + lane;
    const bool mine = lane < A.per_wave && i < A.n;
    double X = 0.0, Y = 0.0, Z = 0.0;
    bool open = false;
    if (mine) {
        X = A.x[i] * A.c.k; Y = A.y[i] * A.c.k; Z = A.z[i] * A.c.k;
        open = atom_open<FIELD>(A.c, A.seed, A.cfg, A.first_atom + (uint64_t)i, X, Y, Z, A.k_first);
        if (!open)
            for (int s = 0; s < A.K; ++s) A.out[i * A.K + s] = __builtin_inf();
    }
    uint64_t todo = __ballot(open);
    if (todo == 0) return;
    const RateRegs R(A.c);
#pragma unroll 1
    while (todo) {
        const int l = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        ionize_atom<FIELD>(A.c, R, A.seed, A.cfg, A.first_atom + (uint64_t)(i0 + l),
                           lane_value(X, l), lane_value(Y, l), lane_value(Z, l), A.k_first, A.K,
                           A.out + (i0 + l) * A.K);
    }
}

// The order for ionize_lane_kernel, most work first: a counting sort by the
// number of states that the rate bound leaves open from the window start, then by
// the peak-field bound in sixteenths of a doubling (the windows, and so the panels
// an atom integrates, grow with it).
constexpr int kIonizeLevels = 372;
constexpr int kIonizeBins = (kMaxStates + 1) * kIonizeLevels;   // 4092
constexpr int kIonizeBlock = 1024;
constexpr int kIonizeChunk = 16 * kIonizeBlock;   // atoms of one block of the last pass

template <int FIELD>
__global__ void __launch_bounds__(kIonizeBlock) ionize_key_kernel(IonizeArgs A, double inv_peak,
                                                                  uint16_t* __restrict__ key,
                                                                  uint32_t* __restrict__ cursor)
{
    __shared__ uint32_t bins[kIonizeBins];
    for (int b = threadIdx.x; b < kIonizeBins; b += kIonizeBlock) bins[b] = 0;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kIonizeBlock + threadIdx.x;
    if (i < A.n) {
        const double X = A.x[i] * A.c.k, Y = A.y[i] * A.c.k, Z = A.z[i] * A.c.k;
        const double b2 = bound2_f64<FIELD>(A.c, X, Y, Z);
        const float depth = -16.0f * log2f((float)(b2 * inv_peak));
        const int level = depth > 0.0f ? (depth < (float)(kIonizeLevels - 1) ? (int)depth : kIonizeLevels - 1)
                                       : (depth <= 0.0f ? 0 : kIonizeLevels - 1);
        int open = 0;
        while (open < A.K && atom_open<FIELD>(A.c, A.seed, A.cfg, A.first_atom + (uint64_t)i, X, Y,
                                              Z, A.k_first + open))
            ++open;
        const int bin = (kMaxStates - open) * kIonizeLevels + level;
        key[i] = (uint16_t)bin;
        atomicAdd(&bins[bin], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kIonizeBins; b += kIonizeBlock)
        if (bins[b]) atomicAdd(&cursor[b], bins[b]);
}

// Counts to first places (one block).
__global__ void __launch_bounds__(kIonizeBlock) ionize_scan_kernel(uint32_t* __restrict__ cursor)
{
    constexpr int kPer = (kIonizeBins + kIonizeBlock - 1) / kIonizeBlock;
    __shared__ uint32_t part[kIonizeBlock];
    uint32_t n[kPer], sum = 0;
    for (int k = 0; k < kPer; ++k) {
        const int b = threadIdx.x * kPer + k;
        sum += n[k] = b < kIonizeBins ? cursor[b] : 0;
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < kIonizeBlock; d *= 2) {
        const uint32_t add = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    uint32_t at = part[threadIdx.x] - sum;
    for (int k = 0; k < kPer; ++k) {
        const int b = threadIdx.x * kPer + k;
        if (b < kIonizeBins) cursor[b] = at;
        at += n[k];
    }
}

__global__ void __launch_bounds__(kIonizeBlock) ionize_place_kernel(
    int64_t n, const uint16_t* __restrict__ key, uint32_t* __restrict__ cursor,
    uint32_t* __restrict__ order)
{
    constexpr int kPer = kIonizeChunk / kIonizeBlock;
    __shared__ uint32_t bins[kIonizeBins], base[kIonizeBins];
    for (int b = threadIdx.x; b < kIonizeBins; b += kIonizeBlock) bins[b] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * kIonizeChunk;
    uint32_t bin[kPer], rank[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t i = lo + k * kIonizeBlock + threadIdx.x;
        bin[k] = i < n ? (uint32_t)key[i] : (uint32_t)kIonizeBins;
        if (bin[k] < kIonizeBins) rank[k] = atomicAdd(&bins[bin[k]], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kIonizeBins; b += kIonizeBlock)
        if (bins[b]) base[b] = atomicAdd(&cursor[b], bins[b]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if (bin[k] < kIonizeBins)
            order[base[bin[k]] + rank[k]] = (uint32_t)(lo + k * kIonizeBlock + threadIdx.x);
}

// Atom order[i] to lane i: neighbours of the order have much the same work.
template <int FIELD>
__global__ void __launch_bounds__(256, IonizeWaves<FIELD>::value) ionize_lane_kernel(IonizeArgs A)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    const int64_t a = (int64_t)A.order[i];
    const RateRegs R(A.c);
    ionize_atom_lane<FIELD>(A.c, R, A.seed, A.cfg, A.first_atom + (uint64_t)a, A.x[a] * A.c.k,
                            A.y[a] * A.c.k, A.z[a] * A.c.k, A.k_first, A.K, A.out + a * A.K);
}

// Wave-cooperative refill: lanes with need == true get consecutive queue
// indices (called by every lane of the wave; -1 for the other lanes).
__device__ inline int64_t queue_take(unsigned long long* queue, bool need)
{
    const uint64_t m = __ballot(need);
    if (m == 0) return -1;
    const int lane = __lane_id();
    const int leader = __ffsll((unsigned long long)m) - 1;
    unsigned long long base = 0;
    if (lane == leader) base = atomicAdd(queue, (unsigned long long)__popcll(m));
    base = __shfl(base, leader);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    return need ? (int64_t)(base + (unsigned long long)rank) : -1;
}

// ---------------------------------------------------------------------------
// Push.  One electron per lane: state (X, u) advanced by classical RK4 with
// fixed step h from its birth to the end of its atom's window (steps start at
// tau0 + n h, the last one ends on the window end).  The fields depend on
// time only through the retarded time D = tau - Z, which the state carries as
// a seventh variable (dD/dtau = 1 - u_z/gamma, D = tau0 - Z0 at birth): RK4
// is linear in its stage slopes, so in exact arithmetic D equals tau - Z at
// every stage, while in floating point the carrier phase is resolved to the
// rounding of D itself rather than that of tau and Z separately (each up to
// ~1e3 over the window).
// ---------------------------------------------------------------------------
template <int FIELD, int AXIS, bool STATED = false, class CFG>
__device__ inline void rhs_f64(const CFG& c, double d, double dl, double X, double Y, double Z,
                               double ux, double uy, double uz, double& dX, double& dY,
                               double& dZ, double& dux, double& duy, double& duz,
                               const fm::Coef& k = fm::kCoef)
{
    const double ig = fm::rsqrt_ge1_f64(1.0 + ux * ux + uy * uy + uz * uz, k);
    dX = ux * ig; dY = uy * ig; dZ = uz * ig;
    if constexpr (FIELD == 1 || FIELD == 3 || FIELD == 5) {
        // radial field: a = (pe X, pe Y, az), b = pb (-Y, X, 0), so
        // a + beta x b = ((pe - beta_z pb) X, (pe - beta_z pb) Y,
        //                 az + pb (beta_x X + beta_y Y))
        double pe, pb, az;
        rp_field_parts_f64<FIELD, true, AXIS>(c, X, Y, Z, d, dl, pe, pb, az, k);
        const double f = fma(-dZ, pb, pe);
        dux = -f * X;
        duy = -f * Y;
        duz = -fma(pb, fma(dY, Y, dX * X), az);
    } else {
        double ax, ay, az, bx, by, bz;
        field_f64<FIELD, true, CFG, false, 0, STATED>(c, X, Y, Z, d + dl, ax, ay, az, bx, by, bz);
        dux = -(ax + dY * bz - dZ * by);
        duy = -(ay + dZ * bx - dX * bz);
        duz = -(az + dX * by - dY * bx);
    }
}

// The state is accumulated with compensated (Kahan) summation: over the
// ~3e4 steps of a trajectory the rounding of plain double accumulation,
// above all of the position, is amplified to more than 1e-8 of the final
// energy for a few electrons in a thousand; the compensation terms cX..cuz
// carry what each addition lost into the next one.
struct ElecF64 {
    double X, Y, Z, ux, uy, uz;
    double D;                                  // retarded time tau - Z
    double cX, cY, cZ, cux, cuy, cuz, cD;
    double h_last;                             // length of the last step
    int32_t left;                              // steps left
};

// Steps from tau0 to the window end taue, 0 when there is none (below 2^31:
// the host limits window / dt to 2e9), and the length of the last one.
__device__ inline int32_t step_count(double tau0, double taue, double h, double& h_last)
{
    const double q = ceil((taue - tau0) / h);
    const int32_t N = q > 0.0 ? (int32_t)q : 0;
    h_last = taue - fma((double)(N - 1), h, tau0);
    return N;
}

constexpr double kLightSpeed = 299792458.0;            // m/s, exact
constexpr double kInvLightSpeed = 1.0 / 299792458.0;

__device__ inline void kahan_add_f64(double& s, double& comp, double v)
{
    const double y = v - comp;
    const double t = s + y;
    comp = (t - s) - y;
    s = t;
}

// Set up an electron born at rest at t0 [s] at atom position (x, y, z) [m].
// Returns false (invalid slot) for a birth more than one step before the
// window start, which also bounds the step count of every lane.
template <class CFG>
__device__ inline bool elec_init(const CFG& c, ElecF64& e, double t0, double x, double y, double z)
{
    e.X = x * c.k; e.Y = y * c.k; e.Z = z * c.k;
    e.ux = e.uy = e.uz = 0.0;
    e.cX = e.cY = e.cZ = e.cux = e.cuy = e.cuz = e.cD = 0.0;
    const double tau0 = t0 * c.omega;
    // D = omega (t0 - z0/c), the quotient z0/c carried with its remainder so
    // that the retarded time is formed to the rounding of its own value
    const double zc = z * kInvLightSpeed;
    const double zr = fma(-zc, kLightSpeed, z);
    e.D = ((t0 - zc) - zr * kInvLightSpeed) * c.omega;
    const double tz = (c.window == 0) ? e.Z : 0.0;
    e.left = 0;
    if (!(tau0 >= tz - c.tb_n - c.hn)) return false;
    e.left = step_count(tau0, tz + c.ta_n, c.hn, e.h_last);
    return true;
}

// One step.  FULL: a step of the full length, which leaves the count of steps
// to the caller; else the one that is due, the last one of its own length.
template <int FIELD, bool FULL = false, bool BATCH = false, class CFG>
__device__ inline void elec_step(const CFG& c, ElecF64& e, const fm::Coef& k)
{
    const double hs = (!FULL && e.left == 1) ? e.h_last : c.hn;
    const double hh = 0.5 * hs;
    double kX, kY, kZ, kx, ky, kz, aX, aY, aZ, ax, ay, az;
    rhs_f64<FIELD, 1, true>(c, e.D, -e.cD, e.X, e.Y, e.Z, e.ux, e.uy, e.uz, kX, kY, kZ, kx, ky, kz, k);
    aX = kX; aY = kY; aZ = kZ; ax = kx; ay = ky; az = kz;
    rhs_f64<FIELD, 0, true>(c, e.D, fma(hh, 1.0 - kZ, -e.cD), e.X + hh * kX, e.Y + hh * kY,
                   e.Z + hh * kZ, e.ux + hh * kx, e.uy + hh * ky, e.uz + hh * kz, kX, kY, kZ, kx,
                   ky, kz, k);
    aX += 2.0 * kX; aY += 2.0 * kY; aZ += 2.0 * kZ;
    ax += 2.0 * kx; ay += 2.0 * ky; az += 2.0 * kz;
    rhs_f64<FIELD, 0, true>(c, e.D, fma(hh, 1.0 - kZ, -e.cD), e.X + hh * kX, e.Y + hh * kY,
                   e.Z + hh * kZ, e.ux + hh * kx, e.uy + hh * ky, e.uz + hh * kz, kX, kY, kZ, kx,
                   ky, kz, k);
    aX += 2.0 * kX; aY += 2.0 * kY; aZ += 2.0 * kZ;
    ax += 2.0 * kx; ay += 2.0 * ky; az += 2.0 * kz;
    rhs_f64<FIELD, 0, true>(c, e.D, fma(hs, 1.0 - kZ, -e.cD), e.X + hs * kX, e.Y + hs * kY,
                   e.Z + hs * kZ, e.ux + hs * kx, e.uy + hs * ky, e.uz + hs * kz, kX, kY, kZ, kx,
                   ky, kz, k);
    const double w6 = hs * (1.0 / 6.0);
    const double sZ = aZ + kZ;
    kahan_add_f64(e.X, e.cX, w6 * (aX + kX));
    kahan_add_f64(e.Y, e.cY, w6 * (aY + kY));
    kahan_add_f64(e.Z, e.cZ, w6 * sZ);
    kahan_add_f64(e.ux, e.cux, w6 * (ax + kx));
    kahan_add_f64(e.uy, e.cuy, w6 * (ay + ky));
    kahan_add_f64(e.uz, e.cuz, w6 * (az + kz));
    // the weighted slopes of D sum to 6 - sZ
    kahan_add_f64(e.D, e.cD, w6 * (6.0 - sZ));
    if (!FULL) --e.left;
}

template <class CFG>
__device__ inline void elec_final(const CFG& c, const ElecF64& e, double& ux, double& uy,
                                  double& uz, double& xf, double& yf, double& zf)
{
    ux = e.ux; uy = e.uy; uz = e.uz;
    xf = e.X * c.inv_k; yf = e.Y * c.inv_k; zf = e.Z * c.inv_k;
}

// ---------------------------------------------------------------------------
// Radiation reaction (Eq. (3)) and the quantum parameter (Eqs. (4)-(5)).  In
// normalized units the gamma^2 Landau-Lifshitz term is
//   du/dtau = -kappa gamma u Q,   Q = (a + beta x b)^2 - (beta . a)^2,
// kappa = (2/3) k r_e, and chi = eta gamma sqrt(Q), eta = hbar omega/(m c^2).
// ElecRR<RR> pushes with the term on (RR) or off and keeps the largest
// gamma^2 Q met at its step starts (chi^2 / eta^2).
// ---------------------------------------------------------------------------
template <bool RR>
struct ElecRR : ElecF64 {
    double g2q;
};

// Right-hand side with the radiation term; returns gamma^2 Q at the state.
template <int FIELD, bool RR, int AXIS, class CFG>
__device__ inline double rhs_rr_f64(const CFG& c, double d, double dl, double X, double Y, double Z,
                                    double ux, double uy, double uz, double& dX, double& dY,
                                    double& dZ, double& dux, double& duy, double& duz,
                                    const fm::Coef& k)
{
    double ax, ay, az, bx, by, bz;
    field_f64<FIELD, true, CFG, true, AXIS>(c, X, Y, Z, d, ax, ay, az, bx, by, bz, dl, k);
    const double ig = fm::rsqrt_ge1_f64(1.0 + ux * ux + uy * uy + uz * uz, k);
    dX = ux * ig; dY = uy * ig; dZ = uz * ig;
    const double fx = ax + (dY * bz - dZ * by);
    const double fy = ay + (dZ * bx - dX * bz);
    const double fz = az + (dX * by - dY * bx);
    // one product of each of the two transverse terms is fused (stated, as in radius2)
    const double bt = FIELD < 20 ? fma(dX, ax, dY * ay) : fma(dY, ay, dX * ax);
    const double ba = fma(dZ, az, bt);
    double q = fx * fx + fy * fy + fz * fz - ba * ba;
    q = q > 0.0 ? q : 0.0;
    dux = -fx; duy = -fy; duz = -fz;
    if (RR) {
        const double s = c.rr_kappa * q / ig;     // kappa gamma Q
        dux -= s * ux; duy -= s * uy; duz -= s * uz;
    }
    return q / (ig * ig);
}

template <class CFG, bool RR>
__device__ inline bool elec_init(const CFG& c, ElecRR<RR>& e, double t0, double x, double y,
                                 double z)
{
    e.g2q = 0.0;
    return elec_init(c, static_cast<ElecF64&>(e), t0, x, y, z);
}

template <int FIELD, bool FULL = false, bool BATCH = false, class CFG, bool RR>
__device__ inline void elec_step(const CFG& c, ElecRR<RR>& e, const fm::Coef& k)
{
    const double hs = (!FULL && e.left == 1) ? e.h_last : c.hn;
    const double hh = 0.5 * hs;
    double kX, kY, kZ, kx, ky, kz, aX, aY, aZ, ax, ay, az;
    const double g2q = rhs_rr_f64<FIELD, RR, 1>(c, e.D, -e.cD, e.X, e.Y, e.Z, e.ux, e.uy, e.uz, kX,
                                             kY, kZ, kx, ky, kz, k);
    e.g2q = g2q > e.g2q ? g2q : e.g2q;
    aX = kX; aY = kY; aZ = kZ; ax = kx; ay = ky; az = kz;
    rhs_rr_f64<FIELD, RR, 0>(c, e.D, fma(hh, 1.0 - kZ, -e.cD), e.X + hh * kX, e.Y + hh * kY,
                          e.Z + hh * kZ, e.ux + hh * kx, e.uy + hh * ky, e.uz + hh * kz, kX, kY,
                          kZ, kx, ky, kz, k);
    aX += 2.0 * kX; aY += 2.0 * kY; aZ += 2.0 * kZ;
    ax += 2.0 * kx; ay += 2.0 * ky; az += 2.0 * kz;
    rhs_rr_f64<FIELD, RR, 0>(c, e.D, fma(hh, 1.0 - kZ, -e.cD), e.X + hh * kX, e.Y + hh * kY,
                          e.Z + hh * kZ, e.ux + hh * kx, e.uy + hh * ky, e.uz + hh * kz, kX, kY,
                          kZ, kx, ky, kz, k);
    aX += 2.0 * kX; aY += 2.0 * kY; aZ += 2.0 * kZ;
    ax += 2.0 * kx; ay += 2.0 * ky; az += 2.0 * kz;
    rhs_rr_f64<FIELD, RR, 0>(c, e.D, fma(hs, 1.0 - kZ, -e.cD), e.X + hs * kX, e.Y + hs * kY,
                          e.Z + hs * kZ, e.ux + hs * kx, e.uy + hs * ky, e.uz + hs * kz, kX, kY,
                          kZ, kx, ky, kz, k);
    const double w6 = hs * (1.0 / 6.0);
    const double sZ = aZ + kZ;
    kahan_add_f64(e.X, e.cX, w6 * (aX + kX));
    kahan_add_f64(e.Y, e.cY, w6 * (aY + kY));
    kahan_add_f64(e.Z, e.cZ, w6 * sZ);
    kahan_add_f64(e.ux, e.cux, w6 * (ax + kx));
    kahan_add_f64(e.uy, e.cuy, w6 * (ay + ky));
    kahan_add_f64(e.uz, e.cuz, w6 * (az + kz));
    kahan_add_f64(e.D, e.cD, w6 * (6.0 - sZ));
    if (!FULL) --e.left;
}


// The configuration where it lies among the kernel's arguments (of the push
// kernels, whose arguments begin with it), read anew at each call: what is
// needed once a step or less does not stay in scalar registers.
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) DevCfg* ColdCfgPtr;
__device__ inline ColdCfgPtr cold_cfg()
{
    ColdCfgPtr p = (ColdCfgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
#else
typedef const DevCfg* ColdCfgPtr;   // host pass: declaration only
__device__ ColdCfgPtr cold_cfg();
#endif

// ---------------------------------------------------------------------------
// Controlled-step push (Sec. 1, Sec. 2.1: fifth-order Runge-Kutta with a
// controlled step, run until the kinetic energy is constant).  Dormand-Prince
// 5(4): seven stages, the fifth-order result carried, the last stage reused
// as the next first one.  One call of elec_step is one attempted step:
//   error = max_i |y5_i - y4_i| / (atol + rtol max(|y_i|, |y5_i|)) over
//           (X, Y, Z, u) in normalized units; accept when <= 1;
//   next step h min(5, max(0.2, 0.9 err^(-1/5))), capped at h_max and at the
//   window end; first step dt;
//   stop at the window end or at the first accepted step end, at least 0.999
//   optical period (2 pi) after the previous check, where gamma changed by at
//   most k_tol relative (the margin keeps steps commensurate with the period
//   from making every check a rounding tie); over the step budget, or when a
//   step's error is not a number, the electron is NaN.
// ---------------------------------------------------------------------------
namespace dp {
constexpr double c2 = 1.0 / 5.0, c3 = 3.0 / 10.0, c4 = 4.0 / 5.0, c5 = 8.0 / 9.0;
constexpr double a21 = 1.0 / 5.0;
constexpr double a31 = 3.0 / 40.0, a32 = 9.0 / 40.0;
constexpr double a41 = 44.0 / 45.0, a42 = -56.0 / 15.0, a43 = 32.0 / 9.0;
constexpr double a51 = 19372.0 / 6561.0, a52 = -25360.0 / 2187.0, a53 = 64448.0 / 6561.0,
                 a54 = -212.0 / 729.0;
constexpr double a61 = 9017.0 / 3168.0, a62 = -355.0 / 33.0, a63 = 46732.0 / 5247.0,
                 a64 = 49.0 / 176.0, a65 = -5103.0 / 18656.0;
// fifth-order weights (b2 = 0, b7 = 0) and fifth minus fourth order
constexpr double b1 = 35.0 / 384.0, b3 = 500.0 / 1113.0, b4 = 125.0 / 192.0,
                 b5 = -2187.0 / 6784.0, b6 = 11.0 / 84.0;
constexpr double e1 = b1 - 5179.0 / 57600.0, e3 = b3 - 7571.0 / 16695.0,
                 e4 = b4 - 393.0 / 640.0, e5 = b5 + 92097.0 / 339200.0,
                 e6 = b6 - 187.0 / 2100.0, e7 = -1.0 / 40.0;
}  // namespace dp

struct ElecDP {
    double y[6];          // X, Y, Z, ux, uy, uz
    double k1[6];         // derivative at y (valid once `fresh` is false)
    double tau, h, taue, g_ref, t_ref;
    int32_t left;         // 1 while the electron runs, 0 when done
    long long acc, rej;
    bool fresh, failed;
};

template <class CFG>
__device__ inline bool elec_init(const CFG& c, ElecDP& e, double t0, double x, double y, double z)
{
    e.y[0] = x * c.k; e.y[1] = y * c.k; e.y[2] = z * c.k;
    e.y[3] = e.y[4] = e.y[5] = 0.0;
    e.tau = t0 * c.omega;
    const double tz = (c.window == 0) ? e.y[2] : 0.0;
    e.taue = tz + c.ta_n;
    e.h = c.hn;
    e.g_ref = 1.0;
    e.t_ref = e.tau;
    e.acc = e.rej = 0;
    e.fresh = true;
    e.failed = false;
    e.left = 0;
    if (!(e.tau >= tz - c.tb_n - c.hn)) return false;
    e.left = (e.taue > e.tau) ? 1 : 0;
    return true;
}

template <int FIELD, int AXIS, class CFG>
__device__ inline void dp_rhs(const CFG& c, double tau, const double* y, double* k,
                              const fm::Coef& co)
{
    rhs_f64<FIELD, AXIS>(c, tau - y[2], 0.0, y[0], y[1], y[2], y[3], y[4], y[5], k[0], k[1], k[2], k[3],
                   k[4], k[5], co);
}

template <int FIELD, bool FULL = false, bool BATCH = false, class CFG>
__device__ inline void elec_step(const CFG& c, ElecDP& e, const fm::Coef& co)
{
    using namespace dp;
    const ColdCfgPtr cold = cold_cfg();
    if (e.fresh) {
        dp_rhs<FIELD, 1>(c, e.tau, e.y, e.k1, co);
        e.fresh = false;
    }
    if (e.acc + e.rej >= cold->ad_max_steps) {
        e.failed = true;
        e.left = 0;
        return;
    }
    double hs = e.h < cold->ad_hmax ? e.h : cold->ad_hmax;
    bool last = false;
    if (hs >= e.taue - e.tau) { hs = e.taue - e.tau; last = true; }
    double k2[6], k3[6], k4[6], k5[6], k6[6], k7[6], yt[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) yt[i] = e.y[i] + hs * (a21 * e.k1[i]);
    dp_rhs<FIELD, 1>(c, e.tau + c2 * hs, yt, k2, co);
#pragma unroll
    for (int i = 0; i < 6; ++i) yt[i] = e.y[i] + hs * (a31 * e.k1[i] + a32 * k2[i]);
    dp_rhs<FIELD, 0>(c, e.tau + c3 * hs, yt, k3, co);
#pragma unroll
    for (int i = 0; i < 6; ++i) yt[i] = e.y[i] + hs * (a41 * e.k1[i] + a42 * k2[i] + a43 * k3[i]);
    dp_rhs<FIELD, 0>(c, e.tau + c4 * hs, yt, k4, co);
#pragma unroll
    for (int i = 0; i < 6; ++i)
        yt[i] = e.y[i] + hs * (a51 * e.k1[i] + a52 * k2[i] + a53 * k3[i] + a54 * k4[i]);
    dp_rhs<FIELD, 0>(c, e.tau + c5 * hs, yt, k5, co);
#pragma unroll
    for (int i = 0; i < 6; ++i)
        yt[i] = e.y[i] + hs * (a61 * e.k1[i] + a62 * k2[i] + a63 * k3[i] + a64 * k4[i] +
                               a65 * k5[i]);
    dp_rhs<FIELD, 0>(c, e.tau + hs, yt, k6, co);
    double y5[6];
#pragma unroll
    for (int i = 0; i < 6; ++i)
        y5[i] = e.y[i] + hs * (b1 * e.k1[i] + b3 * k3[i] + b4 * k4[i] + b5 * k5[i] + b6 * k6[i]);
    dp_rhs<FIELD, 0>(c, e.tau + hs, y5, k7, co);
    double err = 0.0;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const double d = fabs(hs * (e1 * e.k1[i] + e3 * k3[i] + e4 * k4[i] + e5 * k5[i] +
                                    e6 * k6[i] + e7 * k7[i]));
        const double ya = fabs(e.y[i]), yb = fabs(y5[i]);
        const double r = d / (cold->ad_atol + cold->ad_rtol * (ya > yb ? ya : yb));
        err = (r > err || r != r) ? r : err;
    }
    if (err != err) {            // the step produced no number: give up on this electron
        e.failed = true;
        e.left = 0;
        return;
    }
    if (err <= 1.0) {
        e.tau = last ? e.taue : e.tau + hs;
#pragma unroll
        for (int i = 0; i < 6; ++i) { e.y[i] = y5[i]; e.k1[i] = k7[i]; }
        ++e.acc;
        if (last) { e.left = 0; return; }
        if (e.tau - e.t_ref >= 0.999 * (2.0 * 3.14159265358979323846)) {
            const double g = sqrt(1.0 + e.y[3] * e.y[3] + e.y[4] * e.y[4] + e.y[5] * e.y[5]);
            if (fabs(g - e.g_ref) <= cold->ad_ktol * g) { e.left = 0; return; }
            e.g_ref = g;
            e.t_ref = e.tau;
        }
    } else {
        ++e.rej;
    }
    double fac = (err == 0.0) ? 5.0 : 0.9 * pow(err, -0.2);
    fac = fac > 5.0 ? 5.0 : (fac < 0.2 ? 0.2 : fac);
    e.h = hs * fac;
}

template <class CFG>
__device__ inline void elec_final(const CFG& c, const ElecDP& e, double& ux, double& uy,
                                  double& uz, double& xf, double& yf, double& zf)
{
    const double q = __builtin_nan("");
    ux = e.failed ? q : e.y[3]; uy = e.failed ? q : e.y[4]; uz = e.failed ? q : e.y[5];
    xf = e.failed ? q : e.y[0] * c.inv_k;
    yf = e.failed ? q : e.y[1] * c.inv_k;
    zf = e.failed ? q : e.y[2] * c.inv_k;
}

// ---------------------------------------------------------------------------
// Mixed precision: the field and the RK4 stage arithmetic in float; time,
// position and the carrier phase in double.  At each step start the retarded
// time tau - Z is formed in double and reduced to turns in [-1/2, 1/2] (the
// hardware sine/cosine take turns); the four stages then take the transverse
// position, zeta, the phase and the envelope argument as float offsets from
// that start -- the field needs them only to float precision, and the
// retarded time advances by h (1 - beta_z) over a stage of length h.  The
// momentum is kept in float with a Kahan compensation term, the position in
// double.
// ---------------------------------------------------------------------------

// Field arguments at the step start, in float (phase and envelope from the
// double retarded time).
struct MixedBase {
    float X, Y;        // transverse position
    float zeta;        // Z / (k z_r)
    float ph;          // (tau - Z) / (2 pi), reduced to [-1/2, 1/2]
    float s;           // (tau - Z) / (omega tau0)
    float izr, it0;    // 1/(k z_r), 1/(omega tau0)
};

template <class CFG>
__device__ inline MixedBase mixed_base(const CFG& c, double tau, double X, double Y, double Z)
{
    const double d = tau - Z;
    double turns = d * kInvTwoPi;
    turns -= rint(turns);
    MixedBase b;
    b.X = (float)X; b.Y = (float)Y;
    b.zeta = (float)(Z * c.inv_zrn);
    b.ph = (float)turns;
    b.s = (float)(d * c.inv_T0n);
    b.izr = (float)c.inv_zrn;
    b.it0 = (float)c.inv_T0n;
    return b;
}

// Field arguments of a stage at offset hk from the step start, reached with
// the slopes (kX, kY, kZ); dd is the retarded-time offset hk (1 - kZ).
struct MixedArgs {
    float X, Y, zeta, dd, s;
};

template <bool FIRST>
__device__ inline MixedArgs mixed_args(const MixedBase& b, float hk, float kX, float kY, float kZ)
{
    MixedArgs a;
    if constexpr (FIRST) {
        a.X = b.X; a.Y = b.Y; a.zeta = b.zeta; a.dd = 0.f; a.s = b.s;
    } else {
        a.X = fmaf(hk, kX, b.X);
        a.Y = fmaf(hk, kY, b.Y);
        a.zeta = fmaf(hk * kZ, b.izr, b.zeta);
        a.dd = fmaf(-hk, kZ, hk);
        a.s = fmaf(a.dd, b.it0, b.s);
    }
    return a;
}

template <int ORDER, int AXIS, class CFG>
__device__ inline void rp_field_parts_mixed(const CFG& c, const MixedBase& b, const MixedArgs& a,
                                            float& pe, float& pb, float& az)
{
    const float r2 = radius2<AXIS>(a.X, a.Y) * (float)c.inv_w0n2;
    const float zeta = a.zeta;
    const float iD = __builtin_amdgcn_rcpf(1.0f + zeta * zeta);
    const float rD = r2 * iD;
    const float ph = fmaf(a.dd + fmaf(-rD, zeta, (float)c.phi0), (float)kInvTwoPi, b.ph);
    const float g = (float)c.a0 * __builtin_amdgcn_exp2f(-(rD + a.s * a.s) * 1.4426950408889634f);
    const float sn = __builtin_amdgcn_sinf(ph), cs = __builtin_amdgcn_cosf(ph);
    const float gi = g * (iD * iD);
    float PE, PB, EZe;
    rp_brackets<ORDER, float>(gi * cs, gi * sn, zeta, rD, (float)c.e2 * iD, PE, PB, EZe, fm::kCoef);
    pe = (float)c.er_w * PE;
    pb = PB * (float)c.inv_w0n;
    az = (float)c.ez_e * EZe;
}

template <int FIELD, class CFG>
__device__ inline void field_mixed(const CFG& c, const MixedBase& b, const MixedArgs& a,
                                   float& ax, float& ay, float& az, float& bx, float& by,
                                   float& bz)
{
    static_assert(FIELD < 20, "the linearly polarized focus has no mixed form");
    if constexpr (FIELD == 11) {
        ax = (float)c.tE[0]; ay = (float)c.tE[1]; az = (float)c.tE[2];
        bx = (float)c.tB[0]; by = (float)c.tB[1]; bz = (float)c.tB[2];
    } else if constexpr (FIELD == 10) {
        const float ph = fmaf(a.dd + (float)c.phi0, (float)kInvTwoPi, b.ph);
        const float e = (float)c.a0 * __builtin_amdgcn_exp2f(-a.s * a.s * 1.4426950408889634f)
                        * __builtin_amdgcn_cosf(ph);
        ax = e; ay = 0.f; az = 0.f; bx = 0.f; by = e; bz = 0.f;
    } else {
        float pe, pb;
        rp_field_parts_mixed<FIELD, 0>(c, b, a, pe, pb, az);
        ax = pe * a.X; ay = pe * a.Y;
        bx = -pb * a.Y; by = pb * a.X;
        bz = 0.f;
    }
}

template <int FIELD, bool FIRST, int AXIS, class CFG>
__device__ inline void rhs_mixed(const CFG& c, const MixedBase& b, float hk, float& dX, float& dY,
                                 float& dZ, float ux, float uy, float uz, float& dux, float& duy,
                                 float& duz)
{
    // (dX, dY, dZ) come in as the previous stage's slopes and leave as this one's
    const MixedArgs a = mixed_args<FIRST>(b, hk, dX, dY, dZ);
    const float ig = __builtin_amdgcn_rsqf(1.0f + ux * ux + uy * uy + uz * uz);
    dX = ux * ig; dY = uy * ig; dZ = uz * ig;
    if constexpr (FIELD == 1 || FIELD == 3 || FIELD == 5) {
        // radial field: the force from its radial and axial parts, as in rhs_f64
        float pe, pb, az;
        rp_field_parts_mixed<FIELD, AXIS>(c, b, a, pe, pb, az);
        const float f = fmaf(-dZ, pb, pe);
        dux = -f * a.X;
        duy = -f * a.Y;
        duz = -fmaf(pb, fmaf(dY, a.Y, dX * a.X), az);
    } else {
        float ax, ay, az, bx, by, bz;
        field_mixed<FIELD, CFG>(c, b, a, ax, ay, az, bx, by, bz);
        dux = -(ax + dY * bz - dZ * by);
        duy = -(ay + dZ * bx - dX * bz);
        duz = -(az + dX * by - dY * bx);
    }
}

__device__ inline void kahan_add(float& s, float& comp, float v)
{
    const float y = v - comp;
    const float t = s + y;
    comp = (t - s) - y;
    s = t;
}

struct ElecMixed {
    double X, Y, Z, tau0, h_last;
    float ux, uy, uz, cx, cy, cz;
    int32_t n, left;               // steps done and left
};

template <class CFG>
__device__ inline bool elec_init(const CFG& c, ElecMixed& e, double t0, double x, double y, double z)
{
    e.X = x * c.k; e.Y = y * c.k; e.Z = z * c.k;
    e.ux = e.uy = e.uz = 0.f; e.cx = e.cy = e.cz = 0.f;
    e.tau0 = t0 * c.omega;
    const double tz = (c.window == 0) ? e.Z : 0.0;
    e.n = 0;
    e.left = 0;
    if (!(e.tau0 >= tz - c.tb_n - c.hn)) return false;
    e.left = step_count(e.tau0, tz + c.ta_n, c.hn, e.h_last);
    return true;
}

template <int FIELD, bool FULL = false, bool BATCH = false, class CFG>
__device__ inline void elec_step(const CFG& c, ElecMixed& e, const fm::Coef&)
{
    const double h = c.hn;
    const double ta = fma((double)e.n, h, e.tau0);
    const double hsd = (!FULL && e.left == 1) ? e.h_last : h;
    const float hs = (float)hsd, hh = 0.5f * hs;
    const MixedBase b = mixed_base(c, ta, e.X, e.Y, e.Z);
    float kX, kY, kZ, kx, ky, kz, aX, aY, aZ, ax, ay, az;
    rhs_mixed<FIELD, true, BATCH ? 0 : 1>(c, b, 0.f, kX, kY, kZ, e.ux, e.uy, e.uz, kx, ky, kz);
    aX = kX; aY = kY; aZ = kZ; ax = kx; ay = ky; az = kz;
    rhs_mixed<FIELD, false, 0>(c, b, hh, kX, kY, kZ, e.ux + hh * kx, e.uy + hh * ky, e.uz + hh * kz,
                            kx, ky, kz);
    aX += 2.f * kX; aY += 2.f * kY; aZ += 2.f * kZ;
    ax += 2.f * kx; ay += 2.f * ky; az += 2.f * kz;
    rhs_mixed<FIELD, false, 0>(c, b, hh, kX, kY, kZ, e.ux + hh * kx, e.uy + hh * ky, e.uz + hh * kz,
                            kx, ky, kz);
    aX += 2.f * kX; aY += 2.f * kY; aZ += 2.f * kZ;
    ax += 2.f * kx; ay += 2.f * ky; az += 2.f * kz;
    rhs_mixed<FIELD, false, 0>(c, b, hs, kX, kY, kZ, e.ux + hs * kx, e.uy + hs * ky, e.uz + hs * kz,
                            kx, ky, kz);
    const double w6d = hsd * (1.0 / 6.0);
    const float w6 = hs * (1.0f / 6.0f);
    e.X += w6d * (double)(aX + kX); e.Y += w6d * (double)(aY + kY); e.Z += w6d * (double)(aZ + kZ);
    kahan_add(e.ux, e.cx, w6 * (ax + kx));
    kahan_add(e.uy, e.cy, w6 * (ay + ky));
    kahan_add(e.uz, e.cz, w6 * (az + kz));
    ++e.n;
    if (!FULL) --e.left;
}

template <class CFG>
__device__ inline void elec_final(const CFG& c, const ElecMixed& e, double& ux, double& uy,
                                  double& uz, double& xf, double& yf, double& zf)
{
    ux = (double)e.ux; uy = (double)e.uy; uz = (double)e.uz;
    xf = e.X * c.inv_k; yf = e.Y * c.inv_k; zf = e.Z * c.inv_k;
}

// ---------------------------------------------------------------------------
// Persistent push over one configuration, for the controlled-step form, whose
// step counts are not known beforehand, for pushes of few steps, and where the
// ordered push below has no scratch.  A lane whose electron has reached
// its window end writes it out and takes the next slot from a global counter
// (one atomic per wave per refill, ranks from the ballot), so lanes stay busy
// however uneven the step counts are.  Unborn slots are written as NaN when
// taken.
// ---------------------------------------------------------------------------
struct PushIO {
    const double* tb; const double* x0; const double* y0; const double* z0;
    int32_t spa; int64_t n_slots;
    double* ux; double* uy; double* uz; double* xf; double* yf; double* zf;
    unsigned long long* queue;
    double* chi = nullptr;           // largest chi (radiation-reaction push), optional
    double* t_stop = nullptr;        // stop time [s] (controlled-step push), optional
    long long* n_acc = nullptr;      // accepted / rejected steps (controlled-step push)
    long long* n_rej = nullptr;
};

// Electron forms with outputs beyond momentum and position.
template <class E> struct HasExtra { static constexpr bool value = false; };
template <bool RR> struct HasExtra<ElecRR<RR>> { static constexpr bool value = true; };
template <> struct HasExtra<ElecDP> { static constexpr bool value = true; };

template <bool EXTRA>
__device__ inline void write_nan(const PushIO& io, int64_t j)
{
    const double q = __builtin_nan("");
    io.ux[j] = q; io.uy[j] = q; io.uz[j] = q; io.xf[j] = q; io.yf[j] = q; io.zf[j] = q;
    if (EXTRA) {
        if (io.chi) io.chi[j] = q;
        if (io.t_stop) io.t_stop[j] = q;
        if (io.n_acc) io.n_acc[j] = 0;
        if (io.n_rej) io.n_rej[j] = 0;
    }
}

// Per-electron extra outputs: nothing for the plain forms, chi for ElecRR,
// stop time and step counts for ElecDP.
template <class CFG, class E>
__device__ inline void elec_extra(const CFG&, const E&, const PushIO&, int64_t) {}

template <class CFG, bool RR>
__device__ inline void elec_extra(const CFG& c, const ElecRR<RR>& e, const PushIO& io, int64_t j)
{
    if (io.chi) io.chi[j] = c.chi_eta * sqrt(e.g2q);
}

template <class CFG>
__device__ inline void elec_extra(const CFG& c, const ElecDP& e, const PushIO& io, int64_t j)
{
    if (io.t_stop) io.t_stop[j] = e.failed ? __builtin_nan("") : e.tau * c.inv_omega;
    if (io.n_acc) io.n_acc[j] = e.acc;
    if (io.n_rej) io.n_rej[j] = e.rej;
}

// The single-configuration push splits its slots into kQueueParts contiguous
// parts, one counter each (kQueueStride words apart, one 128-byte line per
// counter).  A wave draws from the part of the XCD it runs on (the hardware
// XCC_ID register), so the slots of one part are read and written through one
// XCD's L2, where neighbouring slots share cache lines; lanes that find that
// part used up go on to the next parts in turn.
constexpr int kQueueParts = 8;
constexpr int kQueueStride = 16;
constexpr int kQueueWords = kQueueParts * kQueueStride;

__device__ inline int xcd_id()
{
    // hwreg(HW_REG_XCC_ID, 0, 4): id 20, offset 0, size 4
    return __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & (kQueueParts - 1);
}

// Wave-cooperative refill from the parts of [0, n): lanes with need == true
// get an index, or -1 when every part is used up (a part's counter only
// grows, so a part once used up stays so).
__device__ inline int64_t queue_take_xcd(unsigned long long* queue, int64_t n, bool need)
{
    const int home = xcd_id();
    int64_t got = -1;
    bool want = need;
#pragma unroll 1
    for (int m = 0; m < kQueueParts; ++m) {
        if (__ballot(want) == 0) break;
        const int part = (home + m) & (kQueueParts - 1);
        const int64_t j = queue_take(queue + part * kQueueStride, want);
        const int64_t lo = (n * part) >> 3, hi = (n * (part + 1)) >> 3;   // n / 8 parts
        if (want && j >= 0 && lo + j < hi) {
            got = lo + j;
            want = false;
        }
    }
    return got;
}

// Waves per SIMD each electron form is compiled for (its register budget):
// FP64 RK4 4 (5 needs a few spills and measured no faster), mixed 7 (4 to 7
// within 1%), controlled-step unbounded (six stored stages, 2 waves).  The linear
// focus needs more: order 5 at 4 waves kept 63 doubles in scratch inside the step
// (3e5 slots 436 ms, now 301), order 3 up to 27 registers, some inside it (at 3
// waves, none: the queue form of 6e5 slots of 1000 steps 22.6 -> 21.6 ms, the
// ordered one 19.0 -> 18.8).
template <class E, int FIELD>
struct ElecWaves { static constexpr int value = FIELD == 23 || FIELD == 25 ? 3 : 4; };
template <int FIELD> struct ElecWaves<ElecMixed, FIELD> { static constexpr int value = 7; };
template <int FIELD> struct ElecWaves<ElecDP, FIELD> { static constexpr int value = 1; };
template <bool RR> struct ElecWaves<ElecRR<RR>, 25> { static constexpr int value = 2; };

// Configuration constants of the radial field's step (the members of DevCfg
// that it reads, under the same names).
struct RadialCfg {
    double hn, inv_zrn, inv_w0n2, e2, phi0, inv_T0n, a0_w, er_scale, ez_2, rr_kappa;
};

// What a step reads besides its electron, in registers for the whole kernel.
// A step is bound by instruction issue (one wave on a SIMD takes 5.1 cycles
// for each instruction, scalar ones included; four waves 4.3 for each vector
// one, with scalar ones beside them).  Left to itself the compiler puts a
// literal's two halves into scalar registers at each use: 195 scalar moves and
// 20 moves of spilled scalars in an order-5 step of 841 instructions.  With
// the 38 constants and the 9 of the configuration kept from the start (most in
// scalar pairs; in vector registers where an instruction takes two constants,
// as it can read one scalar operand only, and what no longer fits) the step
// issues 595 vector and 12 scalar instructions, at the same 4 waves.  Measured:
// 8192 slots 45.2 -> 37.0 ms (one wave per SIMD), 1e5 slots 124.3 -> 111.9 ms,
// 2e6 slots 870 -> 838 ms, with radiation reaction 2e4 slots 92.7 -> 77.4 ms.
// The controlled-step form has the vector registers of 2 waves to fill and
// takes most constants there: 1773 -> 1302 instructions in its main block, 2e6
// slots 163.7 -> 145.3 ms.
template <int FIELD, class ELEC>
struct StepRegs {
    static constexpr bool kHold = (FIELD == 1 || FIELD == 3 || FIELD == 5) &&
                                  !std::is_same<ELEC, ElecMixed>::value;
    using Cfg = typename std::conditional<kHold, RadialCfg, DevCfg>::type;
    Cfg c;
    fm::Coef k;
    __device__ inline void set(const DevCfg& d)
    {
        if constexpr (kHold)
            c = RadialCfg{d.hn, d.inv_zrn, d.inv_w0n2, d.e2, d.phi0, d.inv_T0n, d.a0_w, d.er_scale,
                          d.ez_2, d.rr_kappa};
        else
            c = d;
    }
    __device__ inline StepRegs()
    {
        if constexpr (kHold) {
            constexpr bool kWide = std::is_same<ELEC, ElecDP>::value;
            auto keep = [](double& v) {
                if constexpr (kWide) keep_in_vgpr(v); else keep_in_sgpr(v);
            };
            keep_in_vgpr(k.magic);
            keep_in_sgpr(k.log2e); keep_in_sgpr(k.nln2_1); keep_in_sgpr(k.nln2_2);
#pragma unroll
            for (int i = 0; i < 10; ++i) if (i == 8) keep_in_vgpr(k.ex[i]); else keep(k.ex[i]);
            keep_in_sgpr(k.inv_pi); keep_in_sgpr(k.npi_1); keep_in_sgpr(k.npi_2);
            keep_in_vgpr(k.npi_3);
#pragma unroll
            for (int i = 0; i < 7; ++i) if (i == 5) keep_in_vgpr(k.sg[i]); else keep(k.sg[i]);
#pragma unroll
            for (int i = 0; i < 6; ++i) if (i == 4) keep_in_vgpr(k.kp[i]); else keep(k.kp[i]);
            keep_in_vgpr(k.ns2o8); keep_in_vgpr(k.s2);
            keep_in_vgpr(k.c375); keep_in_vgpr(k.c1_0625); keep_in_vgpr(k.c1875);
            keep_in_vgpr(k.c5);
        }
    }
};

struct PushArgs {
    DevCfg c;
    PushIO io;
};

// The kernel's arguments where they lie, read anew at each call: what only the
// refill and the finish of an electron need does not stay in scalar registers.
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) PushArgs* PushArgsPtr;
__device__ inline PushArgsPtr push_args()
{
    PushArgsPtr p = (PushArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
#else
typedef const PushArgs* PushArgsPtr;   // host pass: declaration only
__device__ PushArgsPtr push_args();
#endif

template <int FIELD, class ELEC>
__global__ void __launch_bounds__(256, (ElecWaves<ELEC, FIELD>::value)) push_kernel(PushArgs args)
{
    constexpr bool X = HasExtra<ELEC>::value;
    StepRegs<FIELD, ELEC> R;
    R.set(args.c);
    int64_t idx = -1;
    bool exhausted = false;
    ELEC e;
    e.left = 0;
    while (true) {
        // refill lanes without an electron (unborn slots are consumed here)
        while (true) {
            const bool need = (idx < 0) && !exhausted;
            if (__ballot(need) == 0) break;
            const PushArgsPtr pa = push_args();
            const PushIO io = pa->io;
            const int64_t j = queue_take_xcd(io.queue, io.n_slots, need);
            if (need && j < 0) exhausted = true;
            if (need && j >= 0) {
                const double t0 = io.tb[j];
                if (!(t0 < __builtin_inf())) {
                    write_nan<X>(io, j);
                } else {
                    const DevCfg c = pa->c;
                    const int64_t a = j / io.spa;
                    if (!elec_init(c, e, t0, io.x0[a], io.y0[a], io.z0[a])) {
                        write_nan<X>(io, j);
                        continue;
                    }
                    idx = j;
                    if (e.left <= 0) {
                        elec_final(c, e, io.ux[j], io.uy[j], io.uz[j], io.xf[j], io.yf[j],
                                   io.zf[j]);
                        elec_extra(c, e, io, j);
                        idx = -1;
                    }
                }
            }
        }
        if (__ballot(idx >= 0) == 0) break;
        if (idx >= 0) {
            elec_step<FIELD>(R.c, e, R.k);
            if (e.left == 0) {
                const PushArgsPtr pa = push_args();
                const PushIO io = pa->io;
                const DevCfg c = pa->c;
                elec_final(c, e, io.ux[idx], io.uy[idx], io.uz[idx], io.xf[idx], io.yf[idx],
                           io.zf[idx]);
                elec_extra(c, e, io, idx);
                idx = -1;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Ordered push.  The queue above refills single lanes, so when it runs dry
// every wave is left with a few electrons at any point of their way, and the
// last 1.5 rounds of waves issue for half-empty lanes; and with few electrons,
// some SIMDs hold one wave more than others, which then take that much longer.
// Here the born slots are first put in the order of their step counts (a
// counting sort on kPlanBins bins of N, most steps first), and a wave takes 64
// neighbours of that order, which end together.  Groups of 64 are dealt to W
// waves, a whole number per SIMD: all but the last R < 2 W in whole rounds, one
// launch; those R in time slices, a launch per slice, where the waves go round
// the groups (slice p of the sequence is a step range of group p mod R), so that
// no SIMD has more to do than another.  Between slices the electrons rest in
// memory (128 bytes each, against some 1500 steps).  It waits on nothing but the
// stream's order.  Measured against the queue, with the same step: 1e5 slots
// 111.9 -> 90.9 ms, 2e6 slots in mixed precision 480 -> 450 ms, in double 889 ->
// 884 ms (there the chip lowers its clock with the work in flight, and half-empty
// waves cost little).  The step loop below is what small launches gain by.
// ---------------------------------------------------------------------------
constexpr int kPlanBins = 4096;
constexpr int kPlanBlock = 1024;
constexpr int kPlanChunk = 16 * kPlanBlock;   // slots of one block

struct PushPlan {
    uint32_t born;               // slots in the order
    PlanSplit split;             // waves W, groups in whole rounds, the rest R in slices
    uint32_t slice_steps;
    uint32_t cursor[kPlanBins];  // counts, then the next free place of each bin
};

struct PlanArgs {
    PushPlan* plan;
    uint32_t* order;             // [n_slots]
    uint64_t* state;             // electrons between slices, [word][lane of the rest groups]
    uint32_t simds, max_waves;   // SIMDs of the device, resident waves per SIMD
    double n_max;                // bound of the step counts
};

// Bin of a born slot: its step count in kPlanBins parts of n_max, most first.
__device__ inline uint32_t plan_bin(const DevCfg& c, const PlanArgs& P, double t0, double z)
{
    const double taue = (c.window == 0 ? z * c.k : 0.0) + c.ta_n;
    const double f = (taue - t0 * c.omega) / c.hn * ((double)kPlanBins / P.n_max);
    const double g = fmin(fmax(f, 0.0), (double)(kPlanBins - 1));
    return (uint32_t)(kPlanBins - 1) - (uint32_t)g;
}

// Count the bins; unborn slots are written as NaN here.
template <bool EXTRA>
__global__ void __launch_bounds__(kPlanBlock) plan_count_kernel(DevCfg c, PushIO io, PlanArgs P)
{
    __shared__ uint32_t bins[kPlanBins];
    for (int b = threadIdx.x; b < kPlanBins; b += kPlanBlock) bins[b] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * kPlanChunk;
    const int64_t hi = lo + kPlanChunk < io.n_slots ? lo + kPlanChunk : io.n_slots;
    for (int64_t j = lo + threadIdx.x; j < hi; j += kPlanBlock) {
        const double t0 = io.tb[j];
        if (t0 < __builtin_inf()) atomicAdd(&bins[plan_bin(c, P, t0, io.z0[j / io.spa])], 1u);
        else write_nan<EXTRA>(io, j);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kPlanBins; b += kPlanBlock)
        if (bins[b]) atomicAdd(&P.plan->cursor[b], bins[b]);
}

// Places of the bins, and the plan (one block).
__global__ void __launch_bounds__(kPlanBlock) plan_scan_kernel(PlanArgs P)
{
    constexpr int kPer = kPlanBins / kPlanBlock;
    __shared__ uint32_t part[kPlanBlock];
    __shared__ uint32_t first;
    uint32_t n[kPer], sum = 0;
    for (int i = 0; i < kPer; ++i) sum += n[i] = P.plan->cursor[threadIdx.x * kPer + i];
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < kPlanBlock; d *= 2) {
        const uint32_t add = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    const uint32_t born = part[kPlanBlock - 1];
    const PlanSplit split = plan_split(groups_of(born), P.simds, P.max_waves);
    const uint32_t whole = split.whole;
    if (threadIdx.x == 0) first = 0;
    __syncthreads();
    uint32_t at = part[threadIdx.x] - sum;
    for (int i = 0; i < kPer; ++i) {
        P.plan->cursor[threadIdx.x * kPer + i] = at;
        // the bin that holds the first electron of the rest has its largest count
        if (n[i] && at <= whole * 64 && whole * 64 < at + n[i])
            first = (uint32_t)(threadIdx.x * kPer + i);
        at += n[i];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        PushPlan& p = *P.plan;
        p.born = born;
        p.split = split;
        p.slice_steps = plan_slice_steps((double)(kPlanBins - first) * (P.n_max / (double)kPlanBins),
                                         split.slices);
    }
}

__global__ void __launch_bounds__(kPlanBlock) plan_order_kernel(DevCfg c, PushIO io, PlanArgs P)
{
    __shared__ uint32_t bins[kPlanBins], base[kPlanBins];
    for (int b = threadIdx.x; b < kPlanBins; b += kPlanBlock) bins[b] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * kPlanChunk;
    uint32_t bin[kPlanChunk / kPlanBlock], rank[kPlanChunk / kPlanBlock];
#pragma unroll
    for (int i = 0; i < kPlanChunk / kPlanBlock; ++i) {
        const int64_t j = lo + i * kPlanBlock + threadIdx.x;
        bin[i] = kPlanBins;
        if (j < io.n_slots) {
            const double t0 = io.tb[j];
            if (t0 < __builtin_inf()) {
                bin[i] = plan_bin(c, P, t0, io.z0[j / io.spa]);
                rank[i] = atomicAdd(&bins[bin[i]], 1u);
            }
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kPlanBins; b += kPlanBlock)
        if (bins[b]) base[b] = atomicAdd(&P.plan->cursor[b], bins[b]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPlanChunk / kPlanBlock; ++i)
        if (bin[i] < kPlanBins)
            P.order[base[bin[i]] + rank[i]] = (uint32_t)(lo + i * kPlanBlock + threadIdx.x);
}

// Electrons between slices: word w of every lane side by side.
template <class ELEC>
__device__ inline void put_state(uint64_t* at, size_t stride, const ELEC& e)
{
    static_assert(sizeof(ELEC) % 8 == 0, "whole words");
    uint64_t w[sizeof(ELEC) / 8];
    __builtin_memcpy(w, &e, sizeof(ELEC));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(ELEC) / 8); ++i) at[i * stride] = w[i];
}
template <class ELEC>
__device__ inline void get_state(const uint64_t* at, size_t stride, ELEC& e)
{
    uint64_t w[sizeof(ELEC) / 8];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(ELEC) / 8); ++i) w[i] = at[i * stride];
    __builtin_memcpy(&e, w, sizeof(ELEC));
}

// The number of this lane, computed anew: nothing holds it over a step loop.
__device__ inline uint32_t fresh_lane()
{
    uint32_t lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// Up to `steps` steps of a wave's electrons.  Neighbours in the order have
// nearly the same number of steps left, so all but a few go through a loop with
// no test on any lane, one step length and two steps a turn (the new state then
// need not be copied over the old one); lanes without an electron come along,
// their values are not used.  In double precision a step is 593 instructions
// there instead of 607 and its branches, and one wave on a SIMD issues one every 4.3 cycles
// instead of 5.1 (8192 slots 36.0 -> 29.4 ms, 2e4 slots with radiation reaction
// 76.9 -> 65.5 ms, 2e6 slots 4% faster).  The mixed form, several waves to a
// SIMD, is no faster with it, in twice the code.  Its time depends on where its
// loop (435 instructions, 2.4 KB) lies: with the eight word offsets in a window
// of 32 bytes 6e5 slots took 122 to 141 ms and a sweep of 64 configurations of
// 10,240 slots 149 to 170 ms (150, 149 with one and three words, 161 to 170 with
// the others; order 3 135 to 141, order 1 107 to 109; the double-precision loops
// do not care).  Instruction fetch is the likely reason; no counter was read for
// it.  The alignment and the words below move the loop to the best of the eight.
// The compiler puts the loop's first instructions between, so the number holds
// for the kernels as they stand: after a change to them it is measured again.
// What a lane needs before its steps and after them (its number, its slot) is
// formed anew: held over the loops in registers, these put 28 to 52 bytes a lane
// into scratch (at order 5, 4 and 7 waves).
template <int FIELD, bool BATCH, class CFG, class ELEC>
__device__ inline void run_steps(const CFG& c, ELEC& e, const fm::Coef& k, int32_t steps)
{
    if constexpr (!std::is_same<ELEC, ElecMixed>::value) {
        int32_t least = e.left > 0 ? e.left : 0x7fffffff;
        for (int o = 32; o > 0; o >>= 1) {
            const int32_t other = __shfl_xor(least, o);
            least = other < least ? other : least;
        }
        least = __builtin_amdgcn_readfirstlane(least);
        if (least == 0x7fffffff) return;
        const int32_t full = least - 1 < steps ? least - 1 : steps;
        int32_t n = full;
#pragma unroll 1
        for (; n > 1; n -= 2) {
            elec_step<FIELD, true, BATCH>(c, e, k);
            elec_step<FIELD, true, BATCH>(c, e, k);
        }
        if (n > 0) elec_step<FIELD, true, BATCH>(c, e, k);
        if (e.left > 0) e.left -= full;
        steps -= full;
    }
    if constexpr (std::is_same<ELEC, ElecMixed>::value) {
        if constexpr (BATCH)
            asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
        else
            asm volatile(".p2align 5");
    }
#pragma unroll 1
    for (; steps > 0 && __ballot(e.left > 0) != 0; --steps)
        if (e.left > 0) elec_step<FIELD, false, BATCH>(c, e, k);
}

struct GroupArgs {
    DevCfg c;
    PushIO io;
    PlanArgs P;
    int32_t slice;               // -1: the whole rounds; else the slice launch
};
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) GroupArgs* GroupArgsPtr;
__device__ inline GroupArgsPtr group_args()
{
    GroupArgsPtr p = (GroupArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
#else
typedef const GroupArgs* GroupArgsPtr;   // host pass: declaration only
__device__ GroupArgsPtr group_args();
#endif

template <int FIELD, class ELEC>
__global__ void __launch_bounds__(256, (ElecWaves<ELEC, FIELD>::value)) push_group_kernel(GroupArgs args)
{
    constexpr bool X = HasExtra<ELEC>::value;
    const PushPlan* plan = args.P.plan;
    const uint32_t W = plan->split.waves, whole = plan->split.whole, rest = plan->split.rest;
    const uint32_t wave = (uint32_t)wave_index();
    if (wave >= W) return;
    // whole rounds: groups wave, wave + W, ...; a slice: one group's next steps
    uint32_t group = wave, end = whole;
    int32_t steps = 0x7fffffff;
    bool first = true;
    if (args.slice >= 0) {
        const uint32_t slices = plan->split.slices;
        const PlanTurn t = plan_turn((uint32_t)args.slice, wave, W, rest, slices);
        if (!t.any) return;
        group = whole + t.index;
        end = group + 1;
        first = t.turn == 0;
        if (t.turn + 1 < slices) steps = (int32_t)plan->slice_steps;
    }
    StepRegs<FIELD, ELEC> R;
    R.set(args.c);
    for (; group < end; group += W) {
        ELEC e;
        e.left = 0;
        const uint32_t lane = fresh_lane(), at = group * 64u + lane;
        {
            const GroupArgsPtr ga = group_args();
            const size_t stride = (size_t)rest * 64;
            if (!first) {
                get_state(ga->P.state + (size_t)(group - whole) * 64 + lane, stride, e);
            } else if (at < ga->P.plan->born) {
                const PushIO io = ga->io;
                const DevCfg c = ga->c;
                const int64_t j = (int64_t)ga->P.order[at];
                const int64_t a = j / io.spa;
                if (!elec_init(c, e, io.tb[j], io.x0[a], io.y0[a], io.z0[a])) {
                    write_nan<X>(io, j);
                } else if (e.left <= 0) {
                    elec_final(c, e, io.ux[j], io.uy[j], io.uz[j], io.xf[j], io.yf[j], io.zf[j]);
                    elec_extra(c, e, io, j);
                }
            }
        }
        const bool runs = e.left > 0;
        run_steps<FIELD, false>(R.c, e, R.k, steps);
        {
            const GroupArgsPtr ga = group_args();
            if (runs && e.left == 0) {
                const PushIO io = ga->io;
                const DevCfg c = ga->c;
                const int64_t j = (int64_t)ga->P.order[at];
                elec_final(c, e, io.ux[j], io.uy[j], io.uz[j], io.xf[j], io.yf[j], io.zf[j]);
                elec_extra(c, e, io, j);
            }
            if (steps != 0x7fffffff)
                put_state(ga->P.state + (size_t)(group - whole) * 64 + lane, (size_t)rest * 64, e);
        }
    }
}

// ---------------------------------------------------------------------------
// Histogram.  Each lane computes its bin key and counts it in LDS: all bins
// where they fit, else a table of places that the first bin owns, the rest in
// global memory; the six tallies are ballot-counted per wave.  (Only the
// sweep's binning pass merges the lanes of a wave that share a key.)
// ---------------------------------------------------------------------------
struct HistArgs {
    int32_t nE, nA, angle;
    double lo, width;
    double mec2;  // electron rest energy [MeV]
    double log_mec2, inv_width;   // of the estimate; inv_width NaN: no estimates
};

// atan2 in float, |error| < 1e-6: polynomial 4.4.49 of Abramowitz and Stegun
// (2e-8) in min/max, the rest rounding.  Not both arguments zero.
__device__ inline float angle_estimate(float y, float x)
{
    const float ax = fabsf(x), ay = fabsf(y);
    const float r = fminf(ax, ay) * __builtin_amdgcn_rcpf(fmaxf(ax, ay)), q = r * r;
    float a = 0.0028662257f;
    a = fmaf(a, q, -0.0161657367f);
    a = fmaf(a, q, 0.0429096138f);
    a = fmaf(a, q, -0.0752896400f);
    a = fmaf(a, q, 0.1065626393f);
    a = fmaf(a, q, -0.1420889944f);
    a = fmaf(a, q, 0.1999355085f);
    a = fmaf(a, q, -0.3333314528f);
    a = fmaf(a * q, r, r);
    a = ay > ax ? 1.57079632679f - a : a;
    a = x < 0.0f ? 3.14159265359f - a : a;
    return copysignf(a, y);
}

// Where an electron lies on the two axes, in bins, from float functions: good
// to 0.3e-6 (1 + |log10 K|) in log10 K and 1e-6 in the angle (float rounding
// of the terms, 1 ulp for the hardware's log2, sqrt and rcp).  True if both are
// far enough from a bin edge (three times that) for their floors to be those
// of the exact values.
__device__ inline bool bins_estimate(const HistArgs& H, double up2, double u2, double ux, double uy,
                                     double uz, double& fe, double& fa)
{
    const float v = (float)u2;
    const float r = v * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(1.0f + v) + 1.0f);
    const double lk = fma((double)__builtin_amdgcn_logf(r), 0.30102999566398120, H.log_mec2);
    const double e = (lk - H.lo) * H.inv_width;
    const float t = H.angle == 0
                        ? angle_estimate(__builtin_amdgcn_sqrtf((float)up2), (float)uz) * 0.31830988618f
                        : fmaf(angle_estimate((float)uy, (float)ux), 0.15915494309f, 0.5f);
    const double a = (double)t * (double)H.nA;
    const double me = (1e-6 + 1e-6 * fabs(lk)) * H.inv_width, ma = 1e-6 * (double)H.nA;
    fe = floor(e);
    fa = floor(a);
    return v > 1e-20f && v < 1e20f && up2 > 1e-30 && e - fe > me && e - fe < 1.0 - me && a - fa > ma &&
           a - fa < 1.0 - ma;
}

// Bin key of one electron: >= 0 histogram cell index, or a negative tally code
// -(tally+1) for tallies 2..5; dir returned separately (0 fwd, 1 bwd, -1 none).
// The definition takes a double logarithm, arctangent, two square roots and
// three divisions, some 450 instructions, and bound the histogram; the estimate
// some 90, and 1 in 2000 electrons (256 by 180 bins) is near enough to an edge to
// need the former: 1e7 slots 200 -> 129 us, with 20,000 bins 147 -> 70 us.
__device__ inline int64_t bin_key(const HistArgs& H, double tb, double ux, double uy, double uz,
                                  int& tally, int& dir)
{
#pragma clang fp contract(off)
    dir = -1;
    if (!(tb < __builtin_inf())) { tally = 4; return -1; }
    if (isnan(ux) || isnan(uy) || isnan(uz)) { tally = 5; return -1; }
    const double up2 = ux * ux + uy * uy;
    const double u2 = (ux * ux + uy * uy) + uz * uz;
    dir = (uz > 0.0) ? 0 : 1;
    double fe, fa;
    if (!bins_estimate(H, up2, u2, ux, uy, uz, fe, fa)) {
        const double K = H.mec2 * u2 / (sqrt(1.0 + u2) + 1.0);
        const double pi = 3.14159265358979323846;
        fe = floor((log10(K) - H.lo) / H.width);
        if (H.angle == 0) fa = floor(atan2(sqrt(up2), uz) / pi * (double)H.nA);
        else fa = floor((atan2(uy, ux) + pi) / (2.0 * pi) * (double)H.nA);
    }
    if (!(fe >= 0.0)) { tally = 2; return -1; }
    if (fe >= (double)H.nE) { tally = 3; return -1; }
    int ia = (int)fa;
    ia = ia > H.nA - 1 ? H.nA - 1 : (ia < 0 ? 0 : ia);
    tally = -1;
    return ((int64_t)dir * H.nE + (int64_t)fe) * H.nA + ia;
}

// Add 1 at counter[key] for every lane with key >= 0, merging equal keys
// across the wave first: the lowest pending lane's key is broadcast, the
// lanes holding it are counted by ballot and one atomic adds the count.
// Called by every lane of the wave.
__device__ inline void wave_merge_add(int64_t key, unsigned long long* __restrict__ counter)
{
    const int lane = __lane_id();
    bool pending = key >= 0;
    while (true) {
        const uint64_t act = __ballot(pending);
        if (act == 0) break;
        const int leader = __ffsll((unsigned long long)act) - 1;
        const int64_t lk = __shfl(key, leader);
        const uint64_t same = __ballot(pending && key == lk);
        if (lane == leader) atomicAdd(&counter[lk], (unsigned long long)__popcll(same));
        if (pending && key == lk) pending = false;
    }
}

// Counters of one block.  All bins in the block's LDS where they fit
// (kHistLdsBins); beyond that a direct-mapped table in LDS, where the first bin
// that comes to a place owns it and the others of that place go to global
// memory: a block's 4e4 slots fall into some 8e3 bins, so 9e6 slots leave 2.4e6
// global atomics, spread over all bins alike.  NT tallies are counted per wave
// by ballot while it runs and added to global memory once, at the end: a tally
// is one address for the whole grid, and the two or three atomics on them for
// every 64 slots were what bounded the histograms (1e7 slots, 4.5e5 atomics,
// 5.6 ms whatever the bins).  Now 1e7 pairs take 0.04 ms with the bins in LDS
// (5.7 TB/s), and energies and angles 0.13 ms with 92,160 bins in the table and
// 0.07 ms with 20,000 (4.6 TB/s), where an atomic a slot on the crowded bins in
// global memory takes 1.18 ms; from 2e4 slots on the table is no slower.
constexpr int64_t kHistLdsBins = 8192;     // 32 KiB of 32-bit counters
constexpr int kHistPlaces = 16384;         // 128 KiB of bin numbers and counters
constexpr int kHistBlock = 1024;

template <bool ALL, int NT>
struct BlockCounts {
    unsigned* bins;
    unsigned* owner;
    unsigned* tally;
    unsigned long long* counts;
    unsigned t[NT];
    __device__ inline BlockCounts(unsigned* lds, int64_t nbins, unsigned long long* c)
        : bins(lds + NT), owner(lds + NT + kHistPlaces), tally(lds), counts(c)
    {
        for (int k = 0; k < NT; ++k) t[k] = 0;
        const int words = NT + (ALL ? (int)nbins : kHistPlaces);
        for (int w = threadIdx.x; w < words; w += blockDim.x) lds[w] = 0;
        if constexpr (!ALL)
            for (int w = threadIdx.x; w < kHistPlaces; w += blockDim.x) owner[w] = ~0u;
        __syncthreads();
    }
    __device__ inline void add(int64_t key)
    {
        if (key < 0) return;
        if constexpr (ALL) {
            atomicAdd(&bins[key], 1u);
        } else {
            const unsigned k = (unsigned)key, h = k & (kHistPlaces - 1);   // bins < 2^30
            unsigned o = __hip_atomic_load(&owner[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (o == ~0u) {
                o = atomicCAS(&owner[h], ~0u, k);
                if (o == ~0u) o = k;
            }
            if (o == k) atomicAdd(&bins[h], 1u);
            else atomicAdd(&counts[key], 1ull);
        }
    }
    __device__ inline void tallied(int k, bool hit) { t[k] += (unsigned)__popcll(__ballot(hit)); }
    __device__ inline void finish(int64_t nbins, unsigned long long* tallies)
    {
        if (__lane_id() == 0)
            for (int k = 0; k < NT; ++k) if (t[k]) atomicAdd(&tally[k], t[k]);
        __syncthreads();
        if (threadIdx.x < NT && tally[threadIdx.x])
            atomicAdd(&tallies[threadIdx.x], (unsigned long long)tally[threadIdx.x]);
        const int n = ALL ? (int)nbins : kHistPlaces;
        for (int w = threadIdx.x; w < n; w += blockDim.x)
            if (bins[w])
                atomicAdd(&counts[ALL ? (unsigned)w : owner[w]], (unsigned long long)bins[w]);
    }
};

template <bool ALL>
__global__ void __launch_bounds__(kHistBlock) histogram_kernel(
    HistArgs H, int64_t n, const double* __restrict__ tb, const double* __restrict__ ux,
    const double* __restrict__ uy, const double* __restrict__ uz,
    unsigned long long* __restrict__ counts, unsigned long long* __restrict__ tallies)
{
    extern __shared__ unsigned hist_lds[];
    const int64_t nbins = 2ll * H.nE * H.nA;
    BlockCounts<ALL, 6> B(hist_lds, nbins, counts);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // wave-uniform trip count so every lane takes part in the ballots
    const int64_t base0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63);
    // the next slot is loaded while this one is binned
    double next[4];
    const auto load = [&](int64_t i) {
        if (i < n) { next[0] = tb[i]; next[1] = ux[i]; next[2] = uy[i]; next[3] = uz[i]; }
    };
    load(base0 + __lane_id());
    for (int64_t b = base0; b < n; b += stride) {
        const int64_t i = b + __lane_id();
        const double t = next[0], x = next[1], y = next[2], z = next[3];
        load(i + stride);
        int64_t key = -1;
        int tally = -1, dir = -1;
        if (i < n) key = bin_key(H, t, x, y, z, tally, dir);
        B.add(key);
        // tallies: 0 fwd, 1 bwd, 2 below, 3 above, 4 unborn, 5 NaN
        B.tallied(0, dir == 0);
        B.tallied(1, dir == 1);
        for (int k = 2; k < 6; ++k) B.tallied(k, tally == k);
    }
    B.finish(nbins, tallies);
}

// Two-dimensional forward/backward histogram: pair i adds 1 at
// counts[dir][ia][ib], dir 0 if uz > 0 else 1, ia = floor((a - a_lo)/wa),
// ib likewise; tallies[0] counts pairs outside the ranges, tallies[1] pairs
// with a NaN.  Same arithmetic, without contraction, as the definition.
struct Hist2dArgs {
    double a_lo, wa, b_lo, wb;
    int32_t na, nb;
};

template <bool ALL>
__global__ void __launch_bounds__(kHistBlock) histogram2d_kernel(
    Hist2dArgs H, int64_t n, const double* __restrict__ a, const double* __restrict__ b,
    const double* __restrict__ uz, unsigned long long* __restrict__ counts,
    unsigned long long* __restrict__ tallies)
{
#pragma clang fp contract(off)
    extern __shared__ unsigned hist_lds[];
    const int64_t nbins = 2ll * H.na * H.nb;
    BlockCounts<ALL, 2> B(hist_lds, nbins, counts);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t base0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63);
    for (int64_t w = base0; w < n; w += stride) {
        const int64_t i = w + __lane_id();
        int64_t key = -1;
        int tally = -1;
        if (i < n) {
            const double av = a[i], bv = b[i], u = uz[i];
            if (isnan(av) || isnan(bv) || isnan(u)) {
                tally = 1;
            } else {
                const double fa = floor((av - H.a_lo) / H.wa);
                const double fb = floor((bv - H.b_lo) / H.wb);
                if (fa >= 0.0 && fa < (double)H.na && fb >= 0.0 && fb < (double)H.nb)
                    key = ((int64_t)(u > 0.0 ? 0 : 1) * H.na + (int64_t)fa) * H.nb + (int64_t)fb;
                else
                    tally = 0;
            }
        }
        B.add(key);
        B.tallied(0, tally == 0);
        B.tallied(1, tally == 1);
    }
    B.finish(nbins, tallies);
}

// Per-electron outputs: kinetic energy m c^2 u^2/(gamma + 1) [MeV], polar
// angle atan2(|u_perp|, u_z), azimuth atan2(u_y, u_x), forward flag u_z > 0.
// NaN momenta give NaN energy and angles and flag -1.
__global__ void __launch_bounds__(256) epilogue_kernel(
    int64_t n, double mec2, const double* __restrict__ ux, const double* __restrict__ uy,
    const double* __restrict__ uz, double* __restrict__ K, double* __restrict__ theta,
    double* __restrict__ psi, int32_t* __restrict__ fwd)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x = ux[i], y = uy[i], z = uz[i];
    const double up2 = x * x + y * y;
    const double u2 = up2 + z * z;
    K[i] = mec2 * u2 / (sqrt(1.0 + u2) + 1.0);
    theta[i] = atan2(sqrt(up2), z);
    psi[i] = atan2(y, x);
    fwd[i] = (isnan(x) || isnan(y) || isnan(z)) ? -1 : (z > 0.0 ? 1 : 0);
}

__global__ void zero_u64_kernel(unsigned long long* p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

}  // namespace rpdla
