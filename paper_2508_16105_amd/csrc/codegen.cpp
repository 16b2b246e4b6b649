// codegen.cpp -- emits the mechanism-specific device code (namespace mech):
// NASA-7 thermo, modified-Arrhenius forward rates, equilibrium-constant
// reverse rates, third-body and Lindemann/Troe falloff, the constant-pressure
// source terms (species production rates and heat release, Appendix A
// eqs. (20)-(21)) and their analytic Jacobian, all as straight-line code with
// compile-time species indices so each lane keeps its cell in registers.
//
// The Arrhenius parameters (ln A, b, Ea/R) are read from a device buffer so
// they can change without recompiling; every other constant is a literal.
#include "codegen.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <map>
#include <sstream>

namespace chemmi {
namespace {

std::string lit(double v)
{
    char buf[40];
    std::snprintf(buf, sizeof buf, "%.17g", v);
    std::string s(buf);
    if (s.find_first_of(".eEn") == std::string::npos) s += ".0";
    return s;
}

// C[k] written as a product term for stoichiometric coefficient nu
std::string powc(int k, int nu)
{
    std::string s = "C[" + std::to_string(k) + "]";
    std::string r = s;
    for (int i = 1; i < nu; ++i) r += "*" + s;
    return r;
}

// product of C^nu over a side, optionally skipping one occurrence of species `skip`
// (the derivative of C_m^nu is nu C_m^(nu-1))
std::string side_product(const std::vector<Term>& side, int dsp = -1)
{
    std::string r;
    bool hit = false;
    for (const auto& t : side) {
        int nu = t.nu;
        std::string factor;
        if (t.sp == dsp) {
            hit = true;
            if (nu > 1) factor = lit((double)nu) + (nu - 1 > 0 ? "*" + powc(t.sp, nu - 1) : "");
            else factor = "1.0";
        } else {
            factor = powc(t.sp, nu);
        }
        r += (r.empty() ? "" : "*") + factor;
    }
    if (dsp >= 0 && !hit) return "";
    return r.empty() ? "1.0" : r;
}

// G_k(T) = S_k/R - H_k/RT of species k from its NASA-7 set (host side, for
// the range checks of the generator)
double gibbs_of(const SpeciesData& sp, double T)
{
    const double* a = T < sp.tmid ? sp.lo : sp.hi;
    const double lnT = std::log(T);
    const double s = a[0] * lnT + a[1] * T + a[2] * T * T / 2 + a[3] * T * T * T / 3 + a[4] * T * T * T * T / 4 + a[6];
    const double h = a[0] + a[1] * T / 2 + a[2] * T * T / 3 + a[3] * T * T * T / 4 + a[4] * T * T * T * T / 5 +
                     a[5] / T;
    return s - h;
}

// The reverse rate k_r = k_f / K_c with 1/K_c as a product of per-species
// factors, e^{G_k} for each reactant and e^{-G_k} for each product (times
// (RT/P_atm)^dnu), so a reversible reaction costs a few multiplies instead of
// an exponential of its own (ln K_c = sum_k nu_k G_k + dnu ln(P_atm/RT), the
// standard-state equilibrium constant of the mass-action law).  The factors
// are multiplied reactant, product, reactant, ... ; a reaction keeps the
// exponential of ln k_f - ln K_c when some partial product would leave
// [e^-650, e^650] anywhere on 200 .. 6000 K.
struct SpeciesKc {
    std::vector<bool> product_form;   // per reaction
    std::vector<bool> need_gp, need_gm;   // per species: e^{G_k}, e^{-G_k}
    bool any_dnu = false;
};

std::vector<std::pair<int, int>> kc_factor_order(const ReactionData& r)
{
    // (species, +1 for e^{G}, -1 for e^{-G}), one entry per unit of nu, alternating sides
    std::vector<int> a, b;
    for (const auto& t : r.reac)
        for (int i = 0; i < t.nu; ++i) a.push_back(t.sp);
    for (const auto& t : r.prod)
        for (int i = 0; i < t.nu; ++i) b.push_back(t.sp);
    std::vector<std::pair<int, int>> out;
    for (size_t i = 0; i < std::max(a.size(), b.size()); ++i) {
        if (i < a.size()) out.push_back({a[i], +1});
        if (i < b.size()) out.push_back({b[i], -1});
    }
    return out;
}

SpeciesKc plan_species_kc(const MechanismData& m)
{
    SpeciesKc p;
    const int ns = m.ns(), nr = m.nr();
    p.product_form.assign(nr, false);
    p.need_gp.assign(ns, false);
    p.need_gm.assign(ns, false);
    std::vector<double> temps;
    for (double T = 200.0; T <= 6000.0; T += 5.0) temps.push_back(T);
    for (const auto& sp : m.species) {
        temps.push_back(sp.tmid);
        temps.push_back(std::nextafter(sp.tmid, 0.0));
    }
    const double lim = 650.0;
    for (int j = 0; j < nr; ++j) {
        const auto& r = m.reactions[j];
        if (!r.reversible) continue;
        const auto order = kc_factor_order(r);
        bool ok = true;
        for (double T : temps) {
            double acc = 0.0;
            for (const auto& f : order) {
                const double g = gibbs_of(m.species[f.first], T);
                if (std::fabs(g) > lim) ok = false;
                acc += f.second * g;
                if (std::fabs(acc) > lim) ok = false;
            }
            acc += r.dnu * std::log(kRu * T / kPatm);
            if (std::fabs(acc) > lim) ok = false;
            if (!ok) break;
        }
        p.product_form[j] = ok;
        if (!ok) continue;
        for (const auto& f : order) (f.second > 0 ? p.need_gp : p.need_gm)[f.first] = true;
        if (r.dnu != 0) p.any_dnu = true;
    }
    return p;
}

// c_1 e_1 + c_2 e_2 + ... as source text, led by its first term rather than
// by "0.0 +" (x + 0.0 is not x for x = -0.0, so a compiler must keep such an
// addition); "0.0" when there are no terms
std::string lin_sum(const std::vector<std::pair<double, std::string>>& terms)
{
    if (terms.empty()) return "0.0";
    std::string out;
    for (size_t i = 0; i < terms.size(); ++i) {
        const double c = terms[i].first;
        const std::string& e = terms[i].second;
        if (i == 0) out = c == 1.0 ? e : (c == -1.0 ? "-(" + e + ")" : lit(c) + "*" + e);
        else if (c == 1.0) out += " + " + e;
        else if (c == -1.0) out += " - " + e;
        else if (c < 0.0) out += " - " + lit(-c) + "*" + e;
        else out += " + " + lit(c) + "*" + e;
    }
    return out;
}

// Species no reaction produces or consumes (net coefficient zero in every
// reaction): their rows of the source terms and of the Jacobian are zero.
std::vector<bool> inert_species(const MechanismData& m)
{
    std::vector<bool> inert(m.ns(), true);
    for (const auto& r : m.reactions) {
        std::vector<int> nu(m.ns(), 0);
        for (const auto& t : r.reac) nu[t.sp] -= t.nu;
        for (const auto& t : r.prod) nu[t.sp] += t.nu;
        for (int k = 0; k < m.ns(); ++k)
            if (nu[k]) inert[k] = false;
    }
    return inert;
}

// Structural non-zeros of d wdot_k / d C_m: species k changed by a reaction
// whose rate depends on C_m (a reactant, a product of a reversible reaction,
// or a collision partner with non-zero efficiency).
std::vector<std::vector<bool>> jc_pattern(const MechanismData& m)
{
    const int ns = m.ns();
    std::vector<std::vector<bool>> nz(ns, std::vector<bool>(ns, false));
    for (const auto& r : m.reactions) {
        std::vector<int> nu(ns, 0);
        for (const auto& t : r.reac) nu[t.sp] -= t.nu;
        for (const auto& t : r.prod) nu[t.sp] += t.nu;
        std::vector<bool> dep(ns, false);
        for (const auto& t : r.reac) dep[t.sp] = true;
        if (r.reversible)
            for (const auto& t : r.prod) dep[t.sp] = true;
        if (r.kind == RxnKind::ThirdBody || is_falloff(r.kind))
            for (int k = 0; k < ns; ++k)
                if (r.eff[k] != 0.0) dep[k] = true;
        for (int k = 0; k < ns; ++k)
            if (nu[k])
                for (int mm = 0; mm < ns; ++mm)
                    if (dep[mm]) nz[k][mm] = true;
    }
    return nz;
}

struct Emitter {
    const MechanismData& m;
    std::ostringstream o;
    int ns, nr;
    SpeciesKc kc;
    std::vector<bool> inert;
    std::vector<std::vector<bool>> jnz;

    explicit Emitter(const MechanismData& mm)
        : m(mm), ns(mm.ns()), nr(mm.nr()), kc(plan_species_kc(mm)), inert(inert_species(mm)),
          jnz(jc_pattern(mm)) {}

    // NASA-7 coefficient table, per species and range (0: T < T_mid, 1: T >= T_mid):
    //  [0..4]  cp/R  = c0 + T(c1 + T(c2 + T(c3 + T c4)))          (a1..a5)
    //  [5..8]  H/RT  = c0 + T(c5 + T(c6 + T(c7 + T c8))) + c9/T    (a2/2, a3/3, a4/4, a5/5)
    //  [9]     a6
    //  [10..13] G = S/R - H/RT = c0 lnT + T(c10 + T(c11 + T(c12 + T c13))) + c14 - c9/T
    //           (a2/2, a3/6, a4/12, a5/20), [14] = a7 - a1
    //  [15..18] d(cp/R)/dT = c15 + T(c16 + T(c17 + T c18))            (a2, 2a3, 3a4, 4a5)
    void thermo_table()
    {
        // constant-address-space view: loads through it are scalar (uniform)
        o << "typedef const __attribute__((address_space(4))) double cdbl;\n"
             "// a zero the compiler cannot see through, known to be wave-uniform\n"
             "__device__ __forceinline__ int opaque_zero()\n{\n"
             "  int z;\n  asm volatile(\"s_mov_b32 %0, 0\" : \"=s\"(z));\n"
             "  return __builtin_amdgcn_readfirstlane(z);\n}\n";
        o << "// molar masses: W_k, 1/W_k, R/W_k\n__constant__ double MWTAB[3 * NS] = {";
        for (int t = 0; t < 3; ++t)
            for (int k = 0; k < ns; ++k) {
                const double W = m.species[k].W;
                o << lit(t == 0 ? W : (t == 1 ? 1.0 / W : kRu / W)) << ((t == 2 && k == ns - 1) ? "};\n" : ", ");
            }
        // species enthalpy at 298.15 K (J/kg, the NASA-7 set the kernels choose
        // there): the chemical enthalpy whose release the coupled energy equation sees
        o << "__constant__ double HF298[NS] = {";
        for (int k = 0; k < ns; ++k) {
            const auto& sp = m.species[k];
            const double T = 298.15;
            const double* a = T < sp.tmid ? sp.lo : sp.hi;
            const double hrt = a[0] + a[1] * T / 2 + a[2] * T * T / 3 + a[3] * T * T * T / 4 +
                               a[4] * T * T * T * T / 5 + a[5] / T;
            o << lit(kRu * T * hrt / sp.W) << (k + 1 < ns ? ", " : "};\n");
        }
        o << "__constant__ double THERMO_TMID[NS] = {";
        for (int k = 0; k < ns; ++k) o << lit(m.species[k].tmid) << (k + 1 < ns ? ", " : "};\n");
        o << "__constant__ double THERMO[NS][2][20] = {\n";
        for (int k = 0; k < ns; ++k) {
            o << "  {";
            for (int half = 0; half < 2; ++half) {
                const double* a = half == 0 ? m.species[k].lo : m.species[k].hi;
                const double c[20] = {a[0], a[1], a[2], a[3], a[4], a[1] / 2, a[2] / 3, a[3] / 4, a[4] / 5,
                                      a[5], a[1] / 2, a[2] / 6, a[3] / 12, a[4] / 20, a[6] - a[0],
                                      a[1], 2 * a[2], 3 * a[3], 4 * a[4], 0.0};
                o << "{";
                for (int i = 0; i < 20; ++i) o << lit(c[i]) << (i < 19 ? ", " : "");
                o << "}" << (half == 0 ? ", " : "");
            }
            o << "}" << (k + 1 < ns ? ",\n" : "\n");
        }
        o << "};\n\n";
    }

    // The NASA-7 polynomials at T from the table row c, as power sums over
    // T, T^2, T^3, T^4 (computed once per evaluation) so every step is a
    // multiply-accumulate with the scalar coefficient as a multiplicand (one
    // instruction; a scalar addend would cost two extra moves).
    void poly_body(const std::string& sfx, bool with_dcp)
    {
        o << "        { S a = T4 * c[4]; a = fma(T3, c[3], a); a = fma(T2, c[2], a); a = fma(T, c[1], a);\n"
             "          cpR" << sfx << " = a + c[0]; }\n"
             "        { S a = T4 * c[8]; a = fma(T3, c[7], a); a = fma(T2, c[6], a); a = fma(T, c[5], a);\n"
             "          a = fma(iT, c[9], a); HRT" << sfx << " = a + c[0]; }\n"
             "        { S a = T4 * c[13]; a = fma(T3, c[12], a); a = fma(T2, c[11], a); a = fma(T, c[10], a);\n"
             "          a = fma(lnT, c[0], a); a = fma(-iT, c[9], a); G" << sfx << " = a + c[14]; }\n";
        if (with_dcp)
            o << "        { S a = T3 * c[18]; a = fma(T2, c[17], a); a = fma(T, c[16], a); dcpR" << sfx
              << " = a + c[15]; }\n";
    }

    void thermo_one(const std::string& base, const std::string& sfx, bool with_dcp)
    {
        o << "        { cdbl* c = " << base << ";\n";
        poly_body(sfx, with_dcp);
        o << "        }\n";
    }

    void thermo(bool with_dcp)
    {
        // Group species by T_mid.  When every lane of the wave is on the same
        // side of T_mid the range index is wave-uniform and the coefficients
        // come in by scalar loads; a wave straddling T_mid evaluates both
        // ranges and selects per lane.
        std::vector<double> tmids;
        for (auto& s : m.species) {
            bool seen = false;
            for (double t : tmids) seen = seen || t == s.tmid;
            if (!seen) tmids.push_back(s.tmid);
        }
        for (double tm : tmids) {
            o << "  {\n    const bool below = T < " << lit(tm) << ";\n"
                 "    const bool all_lo = __all(below), all_hi = __all(!below);\n"
                 "    if (all_lo || all_hi) {\n"
                 "      const int r = all_lo ? 0 : 20;\n";
            for (int k = 0; k < ns; ++k) {
                if (m.species[k].tmid != tm) continue;
                const std::string idx = "[" + std::to_string(k) + "]";
                o << "      { cdbl* c = TH + " << k * 40 << " + r;\n";
                poly_body(idx, with_dcp);
                o << "      }\n";
            }
            o << "    } else {\n";
            for (int k = 0; k < ns; ++k) {
                if (m.species[k].tmid != tm) continue;
                const std::string idx = "[" + std::to_string(k) + "]";
                o << "      { S cpR_l, HRT_l, G_l, dcpR_l, cpR_h, HRT_h, G_h, dcpR_h;\n";
                thermo_one("TH + " + std::to_string(k * 40), "_l", with_dcp);
                thermo_one("TH + " + std::to_string(k * 40 + 20), "_h", with_dcp);
                o << "        cpR" << idx << " = below ? cpR_l : cpR_h;\n"
                     "        HRT" << idx << " = below ? HRT_l : HRT_h;\n"
                     "        G" << idx << " = below ? G_l : G_h;\n";
                if (with_dcp) o << "        dcpR" << idx << " = below ? dcpR_l : dcpR_h;\n";
                o << "      }\n";
            }
            o << "    }\n  }\n";
        }
    }

    // state common to rhs and rhs_jac
    void prologue(bool jac)
    {
        // The table and parameter addresses are offset by an opaque zero so the
        // scalar loads of the constants stay inside this evaluation instead of
        // being hoisted out of the substep loop (where ~300 live constants
        // would spill).
        o << "  const int z = opaque_zero();\n"
             "  cdbl* TH = (cdbl*)&THERMO[0][0][0] + z;\n"
             "  cdbl* P = (cdbl*)par + z;\n"
             "  cdbl* MW = (cdbl*)&MWTAB[0] + z;\n"
             "  const S T = y[0];\n"
             "  const S lnT = chem_math::ln(T);\n"
             "  const S iT = chem_math::recip(T);\n"
             "  const S T2 = T * T, T3 = T2 * T, T4 = T2 * T2;\n"
             "  S cpR[NS], HRT[NS], G[NS];\n";
        if (jac) o << "  S dcpR[NS];\n";
        thermo(jac);
        // per-species equilibrium factors e^{G_k}, e^{-G_k} (see SpeciesKc)
        for (int k = 0; k < ns; ++k) {
            if (kc.need_gp[k] || kc.need_gm[k])
                o << "  const S gp" << k << " = chem_math::exp_poly(G[" << k << "]);\n";
            if (kc.need_gm[k]) o << "  const S gm" << k << " = chem_math::recip(gp" << k << ");\n";
        }
        if (kc.any_dnu)
            o << "  const S rtp = T * " << lit(kRu / kPatm) << ";\n"
                 "  const S prt = iT * " << lit(kPatm / kRu) << ";\n";
        o << "  S sig = 0.0;\n";
        for (int k = 0; k < ns; ++k)
            o << "  sig = fma(y[" << 1 + k << "], MW[" << ns + k << "], sig);\n";
        // rho = p / (R T sig); 1/rho = R T sig / p with 1/p given
        o << "  const S Wbar = chem_math::recip(sig);\n"
             "  const S rho = p * Wbar * iT * " << lit(1.0 / kRu) << ";\n"
             "  const S irho = " << lit(kRu) << " * T * sig * ip;\n"
             "  const S ctot = p * iT * " << lit(1.0 / kRu) << ";\n"
             "  S C[NS];\n";
        for (int k = 0; k < ns; ++k)
            o << "  C[" << k << "] = rho * (y[" << 1 + k << "] * MW[" << ns + k << "]);\n";
        o << "  const S lnPRT = " << lit(std::log(kPatm / kRu)) << " - lnT;\n"
             "  S wd[NS];\n"
             "#pragma unroll\n  for (int k = 0; k < NS; ++k) wd[k] = 0.0;\n";
        for (const auto& r : m.reactions)
            if (r.kind == RxnKind::Plog) {
                o << "  const double lnp = chem_math::ln(p);\n";
                break;
            }
    }

    // PLOG: the Arrhenius set at this pressure (pla, plb, ple), linear in ln p
    // between the tabulated pressures and the end sets outside them, written
    // without branches: with w_i = clamp((ln p - ln p_i) / (ln p_i+1 - ln p_i),
    // 0, 1) the set is x_0 + sum_i w_i (x_i+1 - x_i), which telescopes to x_i +
    // w_i (x_i+1 - x_i) inside interval i and to the end sets outside.
    void plog_set(const ReactionData& r)
    {
        const auto& e = r.plog;
        o << "    double pla = " << lit(e[0].lnA) << ", plb = " << lit(e[0].b) << ", ple = " << lit(e[0].EaR)
          << ";\n";
        for (size_t i = 0; i + 1 < e.size(); ++i) {
            o << "    { const double w = fmin(1.0, fmax(0.0, (lnp - " << lit(e[i].lnp) << ") * "
              << lit(1.0 / (e[i + 1].lnp - e[i].lnp)) << "));\n"
                 "      pla = fma(w, " << lit(e[i + 1].lnA - e[i].lnA) << ", pla);\n"
                 "      plb = fma(w, " << lit(e[i + 1].b - e[i].b) << ", plb);\n"
                 "      ple = fma(w, " << lit(e[i + 1].EaR - e[i].EaR) << ", ple); }\n";
        }
    }

    std::string third_body_sum(const ReactionData& r)
    {
        std::string s = "ctot";
        for (int k = 0; k < ns; ++k)
            if (r.eff[k] != 1.0) s += " + " + lit(r.eff[k] - 1.0) + "*C[" + std::to_string(k) + "]";
        return s;
    }

    // mode 0: source terms; 1: source terms and Jacobian; 3: production rates,
    // the Jacobian-transpose product J^T w and the parameter products
    void reaction(int j, int mode)
    {
        const bool jtv = mode == 3;
        const bool jac = mode == 1 || jtv;
        const auto& r = m.reactions[j];
        o << "  { // reaction " << j << "\n";
        // ln k = ln A + b ln T - (Ea/R) / T, one scalar operand per instruction
        o << "    S lnk = lnT * P[" << nr + j << "];\n"
             "    lnk = fma(-iT, P[" << 2 * nr + j << "], lnk);\n"
             "    lnk = lnk + P[" << j << "];\n";
        const bool plog = r.kind == RxnKind::Plog, rev_on = r.reversible;
        if (plog) {
            plog_set(r);
            o << "    lnk = lnk + (lnT * plb - iT * ple + pla);\n";
        }
        const bool pform = rev_on && kc.product_form[j];
        if (pform) {
            // 1/K_c = prod_reac e^{G} prod_prod e^{-G} (RT/P_atm)^dnu
            std::string f;
            for (const auto& t : kc_factor_order(r))
                f += (f.empty() ? "" : " * ") + std::string(t.second > 0 ? "gp" : "gm") + std::to_string(t.first);
            for (int i = 0; i < std::abs(r.dnu); ++i) f += (f.empty() ? "" : " * ") + std::string(r.dnu > 0 ? "rtp" : "prt");
            o << "    const S ikc = " << (f.empty() ? std::string("1.0") : f) << ";\n";
        } else if (rev_on) {
            // ln K_c = sum nu (S/R - H/RT) + dnu ln(P_atm / RT)
            std::vector<std::pair<double, std::string>> lnkc;
            for (auto& t : r.prod) lnkc.push_back({(double)t.nu, "G[" + std::to_string(t.sp) + "]"});
            for (auto& t : r.reac) lnkc.push_back({-(double)t.nu, "G[" + std::to_string(t.sp) + "]"});
            if (r.dnu != 0) lnkc.push_back({(double)r.dnu, "lnPRT"});
            o << "    const S lnKc = " << lin_sum(lnkc) << ";\n";
        }
        const bool falloff = is_falloff(r.kind);
        if (r.kind != RxnKind::Elementary && !plog) o << "    const S Mc = " << third_body_sum(r) << ";\n";
        if (!falloff) {
            o << "    const S kf = chem_math::exp_poly(lnk);\n";
            if (pform) {
                if (jac) o << "    const S kr = kf * ikc;\n";
            } else if (rev_on) {
                o << "    const S kr = chem_math::exp_poly(lnk - lnKc);\n";
            }
        } else {
            // P_r = k0 [M] / k_inf, one exponential for the ratio
            o << "    const S kinf = chem_math::exp_poly(lnk);\n"
                 "    const S lnr0 = " << lit(r.lnA0) << " + " << lit(r.b0) << "*lnT - "
              << lit(r.EaR0) << "*iT - lnk;\n"
                 "    const S r0 = chem_math::exp_poly(lnr0);\n"
                 "    const S Pr = r0 * Mc;\n"
                 "    const bool floored = !(Pr >= 1e-300);\n"
                 // (a branch of the whole wave, with a select in it for the floored lanes:
                 // one of each lane's own would be divergent control flow inside the
                 // step, see ros_step_impl)
                 "    S lgPr = S(-300.0);\n"
                 "    if (__any(!floored)) lgPr = chem_math::lg(Pr);\n"
                 "    const S logPr = floored ? S(-300.0) : lgPr;\n";
            if (r.kind == RxnKind::Troe) {
                o << "    const S e3 = chem_math::exp_neg(-T * " << lit(1.0 / r.T3) << ");\n"
                     "    const S e1 = chem_math::exp_neg(-T * " << lit(1.0 / r.T1) << ");\n";
                o << "    S Fc = " << lit(1.0 - r.alpha) << "*e3 + " << lit(r.alpha) << "*e1;\n";
                if (jac)
                    o << "    S dFc = " << lit(-(1.0 - r.alpha) / r.T3) << "*e3 + "
                      << lit(-r.alpha / r.T1) << "*e1;\n";
                if (r.has_T2) {
                    o << "    const S e2 = chem_math::exp_neg(" << lit(-r.T2) << " * iT);\n"
                         "    Fc += e2;\n";
                    if (jac) o << "    dFc += " << lit(r.T2) << "*iT*iT*e2;\n";
                }
                o << "    const S logFc = chem_math::lg(Fc);\n"
                     "    const S tc = -0.4 - 0.67*logFc;\n"
                     "    const S tn = 0.75 - 1.27*logFc;\n"
                     "    const S tu = logPr + tc;\n"
                     "    const S tden = tn - 0.14*tu;\n"
                     "    const S itden = chem_math::recip(tden);\n"
                     "    const S tx = tu * itden;\n"
                     "    const S iopx2 = chem_math::recip(1.0 + tx*tx);\n"
                     "    const S logF = logFc * iopx2;\n"
                     "    const S Fb = chem_math::exp_neg(" << lit(std::log(10.0)) << " * logF);\n";
                if (jac) {
                    o << "    const S tg = -logFc * 2.0 * tx * (iopx2*iopx2);\n"
                         "    const S dF_dPr = floored ? S(0.0) : tg * tn * (itden*itden);\n"
                         "    const S dF_dFc = iopx2 + tg * (-0.67*tn + 1.27*tu) * (itden*itden);\n"
                         "    const S dlogFc_dT = dFc / (Fc * " << lit(std::log(10.0)) << ");\n";
                }
            } else if (r.kind == RxnKind::Sri) {
                // F = d [a exp(-b/T) + exp(-T/c)]^X T^e with X = 1 / (1 + log10(P_r)^2)
                const double* c = r.sri;
                o << "    const S sea = " << (c[0] != 0.0 ? lit(c[0]) + " * chem_math::exp_poly(" + lit(-c[1]) + " * iT)"
                                                         : std::string("0.0")) << ";\n"
                     "    const S sec = chem_math::exp_poly(-T * " << lit(1.0 / c[2]) << ");\n"
                     "    const S sY = sea + sec;\n"
                     "    const S lnsY = chem_math::ln<true>(sY);\n"
                     "    const S sX = chem_math::recip(1.0 + logPr * logPr);\n"
                     "    const S Fb = chem_math::exp_poly(sX * lnsY + " << lit(c[4]) << " * lnT + " << lit(std::log(c[3]))
                  << ");\n";
                if (jac)
                    o << "    const S dF_dPr = floored ? S(0.0) : lnsY * " << lit(-2.0 / std::log(10.0))
                      << " * logPr * sX * sX;\n"
                         "    const S dF_dFc = 0.0, dlogFc_dT = 0.0;\n"
                         "    const S dlnF_T = sX * (sea * " << lit(c[1]) << " * iT * iT - sec * " << lit(1.0 / c[2])
                      << ") / sY + " << lit(c[4]) << " * iT;\n";
            } else {
                o << "    const S Fb = 1.0;\n";
                if (jac) o << "    const S dF_dPr = 0.0, dF_dFc = 0.0, dlogFc_dT = 0.0;\n";
            }
            o << "    const S ipr1 = chem_math::recip(1.0 + Pr);\n"
                 "    const S kf = kinf * Pr * ipr1 * Fb;\n";
            if (pform) {
                if (jac)
                    o << "    const S iKc = ikc;\n"
                         "    const S kr = kf * iKc;\n";
            } else if (rev_on)
                o << "    const S iKc = chem_math::exp_poly(-lnKc);\n"
                     "    const S kr = kf * iKc;\n";
        }
        if (pform && !jac) {
            // source terms alone: q = k_f (prod_reac C - prod_prod C / K_c),
            // one rounding for the difference
            o << "    const S pf = " << side_product(r.reac) << ";\n"
                 "    const S pr = " << side_product(r.prod) << ";\n"
                 "    const S q = " << (r.kind == RxnKind::ThirdBody ? "Mc * " : "") << "(kf * fma(-ikc, pr, pf));\n";
        } else if (rev_on)
            o << "    const S pf = " << side_product(r.reac) << ";\n"
                 "    const S pr = " << side_product(r.prod) << ";\n"
                 "    const S fwd = kf * pf;\n"
                 "    const S rev = kr * pr;\n";
        else
            o << "    const S pf = " << side_product(r.reac) << ";\n"
                 "    const S fwd = kf * pf;\n";
        const std::string net = rev_on ? "(fwd - rev)" : "fwd";
        if (!(pform && !jac)) {
            if (r.kind == RxnKind::ThirdBody) o << "    const S q = Mc * " << net << ";\n";
            else o << "    const S q = " << (rev_on ? "fwd - rev" : "fwd") << ";\n";
        }
        // production rates
        std::vector<int> nu(ns, 0);
        for (auto& t : r.reac) nu[t.sp] -= t.nu;
        for (auto& t : r.prod) nu[t.sp] += t.nu;
        for (int k = 0; k < ns; ++k)
            if (nu[k]) o << "    wd[" << k << "] = fma(" << lit(nu[k]) << ", q, wd[" << k << "]);\n";
        if (jac) {
            // d ln k_f / dT at fixed [M]; d ln K_c / dT = (sum nu H/RT - dnu) / T
            std::vector<std::pair<double, std::string>> sh;
            for (auto& t : r.prod) sh.push_back({(double)t.nu, "HRT[" + std::to_string(t.sp) + "]"});
            for (auto& t : r.reac) sh.push_back({-(double)t.nu, "HRT[" + std::to_string(t.sp) + "]"});
            if (rev_on)
                o << "    const S dlnKc = (" << lin_sum(sh)
                  << (r.dnu != 0 ? " - " + lit(r.dnu) : std::string()) << ") * iT;\n";
            if (plog)
                o << "    const S dlnkinf = (P[" << nr + j << "] + plb + (P[" << 2 * nr + j << "] + ple)*iT) * iT;\n";
            else
                o << "    const S dlnkinf = (P[" << nr + j << "] + P[" << 2 * nr + j << "]*iT) * iT;\n";
            if (!falloff) {
                o << "    const S dlnkf = dlnkinf;\n";
            } else {
                o << "    const S dlnk0 = (" << lit(r.b0) << " + " << lit(r.EaR0) << "*iT) * iT;\n"
                     "    const S dlnkf = dlnkinf + (ipr1 + dF_dPr) * (dlnk0 - dlnkinf) + ";
                if (r.kind == RxnKind::Sri) o << "dlnF_T;\n";
                else o << lit(std::log(10.0)) << " * dF_dFc * dlogFc_dT;\n";
                o << "    const S dkdM = kinf * r0 * Fb * (ipr1*ipr1 + dF_dPr*ipr1);\n";
            }
            std::string fac = r.kind == RxnKind::ThirdBody ? "Mc * " : "";
            if (rev_on) o << "    const S dqT = " << fac << "(dlnkf * fwd - (dlnkf - dlnKc) * rev);\n";
            else o << "    const S dqT = " << fac << "(dlnkf * fwd);\n";
            // d q / d C_m (dense over the species that enter)
            std::vector<std::string> dq(ns);
            for (int mm = 0; mm < ns; ++mm) {
                std::string t;
                std::string a = side_product(r.reac, mm);
                std::string b = rev_on ? side_product(r.prod, mm) : std::string();
                if (!a.empty()) t += "kf*(" + a + ")";
                if (!b.empty()) t += (t.empty() ? "-" : " - ") + std::string("kr*(") + b + ")";
                if (!t.empty() && r.kind == RxnKind::ThirdBody) t = "Mc*(" + t + ")";
                if (r.kind == RxnKind::ThirdBody && r.eff[mm] != 0.0)
                    t += (t.empty() ? "" : " + ") + lit(r.eff[mm]) + "*" + net;
                if (falloff && r.eff[mm] != 0.0)
                    t += (t.empty() ? "" : " + ") + lit(r.eff[mm]) + "*dMterm";
                dq[mm] = t;
            }
            // k_r = k_f / K_c, so both directions scale with d k_f / d[M]
            if (falloff) o << "    const S dMterm = dkdM*" << (rev_on ? "(pf - iKc*pr)" : "pf") << ";\n";
            for (int mm = 0; mm < ns; ++mm)
                if (!dq[mm].empty()) o << "    const S dq" << mm << " = " << dq[mm] << ";\n";
            if (jtv) {
                // weights of this reaction's rate in w . f (species rows) and in the
                // heat release: wY = sum_k nu_k W_k w_{1+k}, hs = sum_k nu_k H_k/RT;
                // the columns of J^T w collect wY dq_m and hs dq_m; s = sum_m dq_m C_m
                std::vector<std::pair<double, std::string>> ws, hsum, sj;
                for (int k = 0; k < ns; ++k)
                    if (nu[k]) ws.push_back({(double)nu[k], "(MW[" + std::to_string(k) + "]*w[" + std::to_string(1 + k) + "])"});
                for (int k = 0; k < ns; ++k)
                    if (nu[k]) hsum.push_back({(double)nu[k], "HRT[" + std::to_string(k) + "]"});
                for (int mm = 0; mm < ns; ++mm)
                    if (!dq[mm].empty()) sj.push_back({1.0, "dq" + std::to_string(mm) + "*C[" + std::to_string(mm) + "]"});
                o << "    const S wY = " << lin_sum(ws) << ";\n"
                     "    const S hs = " << lin_sum(hsum) << ";\n"
                     "    const S sj = " << lin_sum(sj) << ";\n";
                for (int mm = 0; mm < ns; ++mm)
                    if (!dq[mm].empty())
                        o << "    colA[" << mm << "] = fma(wY, dq" << mm << ", colA[" << mm << "]); colH[" << mm
                          << "] = fma(hs, dq" << mm << ", colH[" << mm << "]);\n";
                o << "    SwY = fma(wY, sj, SwY); HSa = fma(hs, sj, HSa);\n"
                     "    wYT = fma(wY, dqT, wYT); HwT = fma(hs, dqT, HwT);\n";
                // parameter products w . df/dq_j times d q_j / d(ln A, b, Ea)
                o << "    const S wsum = wY * irho - w[0] * (" << lit(kRu) << " * T) * hs * rcpinv;\n";
                if (falloff) o << "    const S qA = q * (Pr * ipr1 - dF_dPr);\n";
                else o << "    const S qA = q;\n";
                o << "    const S g = wsum * qA;\n"
                     "    chem_math::param_acc(gA[" << j << " * GS], g, gsc);\n"
                     "    chem_math::param_acc(gb[" << j << " * GS], g * lnT, gsc);\n"
                     "    chem_math::param_acc(gE[" << j << " * GS], g * (-iT * " << lit(1.0 / kRu) << "), gsc);\n  }\n";
                return;
            }
            for (int k = 0; k < ns; ++k) {
                if (!nu[k]) continue;
                for (int mm = 0; mm < ns; ++mm)
                    if (!dq[mm].empty())
                        o << "    J[" << 1 + k << "][" << 1 + mm << "] = fma(" << lit(nu[k]) << ", dq" << mm
                          << ", J[" << 1 + k << "][" << 1 + mm << "]);\n";
                o << "    J[" << 1 + k << "][0] = fma(" << lit(nu[k]) << ", dqT, J[" << 1 + k << "][0]);\n";
            }
        }
        o << "  }\n";
    }

    void rhs_tail()
    {
        // 1/(rho cp) = T sig / (p cpm)
        o << "  const S icpm = chem_math::recip(cpm);\n"
             "  const S rcpinv = T * sig * ip * icpm;\n";
        // (species no reaction changes have wdot = 0: no terms, zero rows)
        o << "  S hw = 0.0;\n";
        for (int k = 0; k < ns; ++k)
            if (!inert[k]) o << "  hw = fma(HRT[" << k << "], wd[" << k << "], hw);\n";
        for (int k = 0; k < ns; ++k) {
            if (inert[k]) o << "  f[" << 1 + k << "] = 0.0;\n";
            else o << "  f[" << 1 + k << "] = MW[" << k << "] * (irho * wd[" << k << "]);\n";
        }
        o << "  f[0] = -" << lit(kRu) << " * T * hw * rcpinv;\n";
    }

    void cp_sum(bool jac)
    {
        o << "  S cpm = 0.0;\n";
        for (int k = 0; k < ns; ++k)
            o << "  cpm = fma(cpR[" << k << "], y[" << 1 + k << "] * MW[" << ns + k << "], cpm);\n";
        o << "  const S cp = " << lit(kRu) << " * cpm;\n";
        if (jac) {
            o << "  S dcpm = 0.0;\n";
            for (int k = 0; k < ns; ++k)
                o << "  dcpm = fma(dcpR[" << k << "], y[" << 1 + k << "] * MW[" << ns + k << "], dcpm);\n";
            o << "  const S dcp = " << lit(kRu) << " * dcpm;\n";
        }
    }

    void chain_rule()
    {
        // J holds Jc_km = d wdot_k / d C_m (at fixed T) in its species block and
        // wT_k = d wdot_k / dT (at fixed C) in column 0 of the species rows.
        // With S_k = sum_l Jc_kl C_l:
        //   J_km = (W_k/W_m) Jc_km + (Wbar/W_m)(f_k - W_k S_k / rho)
        //   J_k0 = (W_k / rho)(wT_k - S_k / T) + f_k / T
        //   J_0m = -R T (rho HJ_m - Wbar HS) / (W_m rho cp) - f_T (cp_m / cp - Wbar / W_m)
        //   J_00 = -R (cpw + T HwT - HS) / (rho cp) - f_T (dcp / cp - 1/T)
        // where HJ_m = sum_k H_k/RT Jc_km, HS = sum_k H_k/RT S_k, HwT = sum_k H_k/RT wT_k,
        // cpw = sum_k cp_k/R wdot_k.
        // (sums run over the structural non-zeros of Jc only: a literal zero
        // times a value is not folded away by the compiler, as the value could
        // be infinite; rows of species no reaction changes are zero)
        o << "  S Sk[NS];\n";
        for (int k = 0; k < ns; ++k) {
            std::vector<std::pair<double, std::string>> t;
            for (int l = 0; l < ns; ++l)
                if (jnz[k][l])
                    t.push_back({1.0, "J[" + std::to_string(1 + k) + "][" + std::to_string(1 + l) + "]*C[" + std::to_string(l) + "]"});
            o << "  Sk[" << k << "] = " << lin_sum(t) << ";\n";
        }
        o << "  S HS = 0.0, HwT = 0.0, cpw = 0.0;\n";
        for (int k = 0; k < ns; ++k)
            if (!inert[k])
                o << "  HS = fma(HRT[" << k << "], Sk[" << k << "], HS); HwT = fma(HRT[" << k << "], J[" << 1 + k
                  << "][0], HwT); cpw = fma(cpR[" << k << "], wd[" << k << "], cpw);\n";
        o << "  const S fT = f[0];\n"
             "  const S RT = " << lit(kRu) << " * T;\n"
             "  const S icp = icpm * " << lit(1.0 / kRu) << ";\n";
        // (the columns of species no reaction changes last, and only if asked for:
        // a step's unknowns are the others)
        std::vector<int> cols;
        for (int pass = 0; pass < 2; ++pass)
            for (int mm = 0; mm < ns; ++mm)
                if (inert[mm] == (pass == 1)) cols.push_back(mm);
        const std::string only = "if constexpr (INERT) ";
        for (int mm : cols) {
            std::vector<std::pair<double, std::string>> hj;
            for (int k = 0; k < ns; ++k)
                if (jnz[k][mm])
                    hj.push_back({1.0, "HRT[" + std::to_string(k) + "]*J[" + std::to_string(1 + k) + "][" + std::to_string(1 + mm) + "]"});
            o << "  " << (inert[mm] ? only : "") << "{ S HJ = " << lin_sum(hj) << ";\n"
                 "    S t = fma(rho, HJ, -Wbar*HS) * (-RT * rcpinv);\n"
                 "    S u = fma(cpR[" << mm << "], icp * " << lit(kRu) << ", -Wbar);\n"
                 "    J[0][" << 1 + mm << "] = fma(-fT, u, t) * MW[" << ns + mm << "]; }\n";
        }
        o << "  J[0][0] = -" << lit(kRu) << " * (cpw + T*HwT - HS) * rcpinv - fT * (dcp * icp - iT);\n";
        for (int k = 0; k < ns; ++k) {
            if (inert[k]) continue;   // a zero row
            // J_km = (1/W_m)(W_k Jc_km + Wbar g_k), g_k = f_k - W_k S_k / rho
            o << "  { const S g = fma(-MW[" << k << "], Sk[" << k << "] * irho, f[" << 1 + k << "]);\n"
                 "    const S wg = Wbar * g;\n";
            for (int mm : cols)
                o << "    " << (inert[mm] ? only : "") << "J[" << 1 + k << "][" << 1 + mm << "] = fma(J[" << 1 + k << "]["
                  << 1 + mm << "], MW[" << k << "], wg) * MW[" << ns + mm << "];\n";
            o << "    J[" << 1 + k << "][0] = fma(MW[" << k << "] * irho, J[" << 1 + k << "][0] - Sk[" << k
              << "] * iT, f[" << 1 + k << "] * iT); }\n";
        }
    }

    std::string run()
    {
        o << "// generated mechanism code: " << m.name << " (" << ns << " species, " << nr << " reactions)\n"
          << "namespace mech {\n"
          << "constexpr int NS = " << ns << ";\n"
          << "constexpr int NR = " << nr << ";\n"
          << "constexpr int N = NS + 1;\n"
          << "constexpr double RU = " << lit(kRu) << ";\n";
        // elimination order of the step matrix: T and the species some reaction
        // changes first, then the species no reaction changes, whose rows of
        // M = I/(gamma h) - J are the diagonal alone
        {
            std::vector<int> perm{0};
            for (int k = 0; k < ns; ++k)
                if (!inert[k]) perm.push_back(1 + k);
            const int nact = (int)perm.size();
            for (int k = 0; k < ns; ++k)
                if (inert[k]) perm.push_back(1 + k);
            o << "constexpr int NACT = " << nact << ";   // components with a non-trivial row\n"
              << "constexpr int PERM[N] = {";
            for (int i = 0; i <= ns; ++i) o << perm[i] << (i < ns ? ", " : "};\n\n");
        }
        // source terms only
        thermo_table();
        o << "template <class S>\n__device__ __forceinline__ void rhs(const double* __restrict__ par, double p, "
             "double ip, const S (&y)[N], S (&f)[N])\n{\n";
        prologue(false);
        for (int j = 0; j < nr; ++j) reaction(j, 0);
        cp_sum(false);
        rhs_tail();
        o << "}\n\n";
        // source terms and Jacobian
        o << "// INERT: with the columns of species no reaction changes\n"
             "template <class S, bool INERT = false>\n__device__ __forceinline__ void rhs_jac(const double* __restrict__ par, double p, "
             "double ip, const S (&y)[N], S (&f)[N], S (&J)[N][N])\n{\n";
        o << "#pragma unroll\n  for (int i = 0; i < N; ++i)\n#pragma unroll\n    for (int j = 0; j < N; ++j) J[i][j] = 0.0;\n";
        prologue(true);
        for (int j = 0; j < nr; ++j) reaction(j, 1);
        cp_sum(true);
        rhs_tail();
        chain_rule();
        o << "}\n\n";
        // v = J(y)^T w and the parameter products in one pass, without forming J:
        // every entry of J is assembled from per-reaction partials, so J^T w
        // needs only per-reaction weights and two column sums (see chain_rule):
        //   v_{1+m} = (colA_m + Wbar (w.f_Y - SwY/rho)) / W_m + w_0 J_{0,1+m}
        //   v_0     = (wYT - SwY/T)/rho + (w.f_Y)/T + w_0 J_00
        // with colA_m = sum_j wY_j dq_j/dC_m, colH_m = sum_j hs_j dq_j/dC_m (= HJ_m),
        // SwY = sum_j wY_j s_j, HS = sum_j hs_j s_j, wYT = sum_j wY_j dq_j/dT,
        // HwT = sum_j hs_j dq_j/dT, s_j = sum_m dq_j/dC_m C_m.
        // (the parameter products go to double accumulators, scaled by gsc; for
        // a dual S only their tangent is added, see chem_math::param_acc; GS is
        // the accumulators' element stride)
        o << "template <class S, int GS = 1>\n__device__ __forceinline__ void jtv_param(const double* __restrict__ par, double p, "
             "double ip, const S (&y)[N], const double (&w)[N], S (&v)[N], double* __restrict__ gA, "
             "double* __restrict__ gb, double* __restrict__ gE, double gsc)\n{\n";
        prologue(true);
        cp_sum(true);
        o << "  const S icpm = chem_math::recip(cpm);\n"
             "  const S rcpinv = T * sig * ip * icpm;\n"
             "  S colA[NS], colH[NS];\n"
             "#pragma unroll\n  for (int k = 0; k < NS; ++k) { colA[k] = 0.0; colH[k] = 0.0; }\n"
             "  S SwY = 0.0, HSa = 0.0, wYT = 0.0, HwT = 0.0;\n";
        for (int j = 0; j < nr; ++j) reaction(j, 3);
        o << "  S hw = 0.0, Wf = 0.0, cpw = 0.0;\n";
        for (int k = 0; k < ns; ++k)
            if (!inert[k])
                o << "  hw = fma(HRT[" << k << "], wd[" << k << "], hw); cpw = fma(cpR[" << k << "], wd[" << k
                  << "], cpw); Wf = fma(w[" << 1 + k << "], MW[" << k << "] * (irho * wd[" << k << "]), Wf);\n";
        o << "  const S fT = -" << lit(kRu) << " * T * hw * rcpinv;\n"
             "  const S RT = " << lit(kRu) << " * T;\n"
             "  const S icp = icpm * " << lit(1.0 / kRu) << ";\n"
             "  const S SwYg = Wf - irho * SwY;\n"
             "  const S wg = Wbar * SwYg;\n";
        for (int mm = 0; mm < ns; ++mm)
            o << "  { S t = fma(rho, colH[" << mm << "], -Wbar*HSa) * (-RT * rcpinv);\n"
                 "    S u = fma(cpR[" << mm << "], icp * " << lit(kRu) << ", -Wbar);\n"
                 "    const S J0m = fma(-fT, u, t) * MW[" << ns + mm << "];\n"
                 "    v[" << 1 + mm << "] = fma(colA[" << mm << "] + wg, MW[" << ns + mm << "], w[0] * J0m); }\n";
        o << "  const S J00 = -" << lit(kRu) << " * (cpw + T*HwT - HSa) * rcpinv - fT * (dcp * icp - iT);\n"
             "  v[0] = fma(irho, wYT - SwY * iT, fma(iT, Wf, w[0] * J00));\n";
        o << "}\n\n}  // namespace mech\n";
        return o.str();
    }
};

}  // namespace

int active_unknowns(const MechanismData& m)
{
    const std::vector<bool> inert = inert_species(m);
    return 1 + (int)std::count(inert.begin(), inert.end(), false);
}

std::string generate_mechanism_source(const MechanismData& m) { return Emitter(m).run(); }

namespace {

// number of species slots of a side (a coefficient of 2 takes two slots)
int molecularity(const std::vector<Term>& side)
{
    int n = 0;
    for (const auto& t : side) n += t.nu;
    return n;
}

// species whose third-body efficiency in r is not 1
std::vector<int> partners(const ReactionData& r)
{
    std::vector<int> p;
    for (size_t k = 0; k < r.eff.size(); ++k)
        if (r.eff[k] != 1.0) p.push_back((int)k);
    return p;
}

bool has_third_body(RxnKind k) { return k == RxnKind::ThirdBody || is_falloff(k); }

}  // namespace

WideLayout wide_layout(const MechanismData& m)
{
    WideLayout w;
    const int ns = m.ns(), nr = m.nr();
    w.G = 0;
    int maxt = 1, n_eff = 0, n_plog = 0;
    for (const auto& r : m.reactions) {
        maxt = std::max<int>(maxt, (int)std::max(r.reac.size(), r.prod.size()));
        for (const auto* side : {&r.reac, &r.prod})
            for (const auto& t : *side)
                if (t.nu > 3) return w;
        if (r.dnu < -4 || r.dnu > 3) return w;   // the packed reaction words' field widths
        if (r.kind == RxnKind::Plog) ++n_plog;
        else if (r.kind != RxnKind::Elementary) ++n_eff;
    }
    if (ns + 1 > 64 || maxt > 3 || n_eff > 511 || n_plog > 511 || nr > 65535) return w;
    w.G = 16;
    const std::vector<bool> inert = inert_species(m);
    w.na = (int)std::count(inert.begin(), inert.end(), false);
    const int ni = ns - w.na, nact = w.na + 1;
    w.r = (nact + 15) / 16;
    w.ri = (ni + 1 + 15) / 16;
    w.molr = w.molp = 1;
    for (const auto& r : m.reactions) {
        w.molr = std::max(w.molr, molecularity(r.reac));
        w.molp = std::max(w.molp, molecularity(r.prod));
        if (has_third_body(r.kind)) {
            ++w.ntb;
            w.maxp = std::max<int>(w.maxp, (int)partners(r).size());
        }
    }
    const SpeciesKc kc = plan_species_kc(m);
    for (int j = 0; j < nr; ++j)
        if (m.reactions[j].reversible && !kc.product_form[j]) w.lnkc = true;
    // the scratch of a cell, as the device code lays it out
    const int sp = ns + 1, nrw = nr + 1;
    const int l_a = (w.lnkc ? 5 : 4) * sp;
    const int fwd = l_a + std::max(16 * w.r, std::max(5, w.molr + w.molp) * nrw + w.ntb * (1 + w.maxp));
    // cells 16 doubles apart modulo the 64 banks, so two cells' rows do not collide
    auto pad = [](int n) { return n + (48 - n % 32) % 32; };
    w.lds_cell = pad(fwd);
    const int words = (w.molr + 3) / 4 + (w.molp + 3) / 4 + 1, npt = 16 * (w.r + w.ri);
    w.table = 3 * nr + 38 * npt + (11 + w.maxp) * w.ntb + (words * nr + w.maxp * w.ntb + 1) / 2;
    // a workgroup is four waves of four cells that share the tables; fewer waves,
    // then fewer cells a wave, where that does not fit the 160 KB of LDS
    while (w.wpb * w.cpw > 1 && (size_t)(w.table + w.wpb * w.cpw * w.lds_cell) * sizeof(double) > 160 * 1024)
        (w.wpb > 1 ? w.wpb : w.cpw) /= 2;
    return w;
}

std::string generate_wide_source(const MechanismData& m, const WideLayout& w)
{
    Emitter e(m);
    std::ostringstream& o = e.o;
    const int ns = m.ns(), nr = m.nr(), na = w.na, ni = ns - na, nact = na + 1;
    const int npt = 16 * (w.r + w.ri);
    // position order of the species: changed by some reaction, then the others
    std::vector<int> ord, inv(ns);
    for (int pass = 0; pass < 2; ++pass)
        for (int k = 0; k < ns; ++k)
            if (e.inert[k] == (pass == 1)) ord.push_back(k);
    for (int q = 0; q < ns; ++q) inv[ord[q]] = q;
    // position -> species (-1: T's position or none)
    std::vector<int> pspec(npt, -1);
    for (int q = 0; q < na; ++q) pspec[1 + q] = ord[q];
    for (int q = 0; q < ni; ++q) pspec[16 * w.r + q] = ord[na + q];
    int maxdnu = 0;
    bool sri = false, irrev = false;
    for (const auto& r : m.reactions) {
        if (r.reversible) maxdnu = std::max(maxdnu, std::abs(r.dnu));
        sri = sri || r.kind == RxnKind::Sri;
        irrev = irrev || !r.reversible;
    }
    // reactions in evaluation order: those with extra terms first (PLOG, SRI,
    // Troe, Lindemann, third body), so that as few rounds of 16 lanes as can be
    // hold any, then the elementary ones
    std::vector<int> order;
    for (int kind = 5; kind >= 0; --kind)
        for (int j = 0; j < nr; ++j)
            if ((int)m.reactions[j].kind == kind) order.push_back(j);
    int nfull = 0;
    for (const auto& r : m.reactions) nfull += r.kind != RxnKind::Elementary;
    const int full_rounds = (nfull + 15) / 16;
    const bool has_plog = std::any_of(m.reactions.begin(), m.reactions.end(),
                                      [](const ReactionData& r) { return r.kind == RxnKind::Plog; });
    const bool has_troe = std::any_of(m.reactions.begin(), m.reactions.end(),
                                  [](const ReactionData& r) { return r.kind == RxnKind::Troe; });
    const bool one_tmid = std::all_of(m.species.begin(), m.species.end(),
                                      [&](const auto& s) { return s.tmid == m.species[0].tmid; });
    auto yn = [](bool b) { return b ? "true" : "false"; };
    o << "// generated mechanism tables (wave-cooperative form): " << m.name << " (" << ns << " species, " << nr
      << " reactions)\n"
      << "namespace mech {\n"
      << "constexpr int NS = " << ns << ";\n"
      << "constexpr int NR = " << nr << ";\n"
      << "constexpr int N = NS + 1;\n"
      << "constexpr int NA = " << na << ", NI = " << ni << ", NACT = " << nact
      << ";   // species some reaction changes, the others; unknowns of a step\n"
      << "constexpr int R = " << w.r << ", RI = " << w.ri << ", NPT = " << npt << ";   // positions a lane, in all\n"
      << "constexpr int MOLR = " << w.molr << ", MOLP = " << w.molp << ", MAXDNU = " << maxdnu << ";\n"
      << "constexpr int NTB = " << w.ntb << ", MAXP = " << w.maxp << ";\n"
      << "constexpr int FULL_ROUNDS = " << full_rounds << ";   // leading rounds with slots other than elementary\n"
      << "constexpr int LDS_CELL = " << w.lds_cell << ";   // doubles of scratch per cell\n"
      << "constexpr int CPW = " << w.cpw << ";   // cells per wave\n"
      << "constexpr int WPS = " << w.waves_per_simd() << ";   // waves per SIMD the registers are shared by\n"
      << "constexpr double RU = " << lit(kRu) << ";\n"
      << "constexpr double RU_PATM = " << lit(kRu / kPatm) << ", PATM_RU = " << lit(kPatm / kRu) << ";\n"
      << "constexpr double LN_PATM_R = " << lit(std::log(kPatm / kRu)) << ";\n"
      << "constexpr double LN10 = " << lit(std::log(10.0)) << ";\n"
      << "// reaction forms present (the kernels leave out the code of the absent ones)\n"
         "constexpr bool HAS_PLOG = " << yn(has_plog) << ", HAS_SRI = " << yn(sri) << ", HAS_IRREV = " << yn(irrev)
      << ", HAS_LNKC = " << yn(w.lnkc) << ", HAS_TROE = " << yn(has_troe) << ";\n"
      << "constexpr bool ONE_TMID = " << yn(one_tmid) << ";   // one temperature parts every species' ranges\n"
      << "constexpr double TMID = " << lit(m.species[0].tmid) << ";\n";
    e.thermo_table();
    auto ints = [&](const std::string& decl, const std::vector<int>& v) {
        o << decl << "[" << std::max<size_t>(v.size(), 1) << "] = {";
        if (v.empty()) o << "0";
        for (size_t i = 0; i < v.size(); ++i) o << v[i] << (i + 1 < v.size() ? ", " : "");
        o << "};\n";
    };
    auto dbls = [&](const std::string& decl, const std::vector<double>& v) {
        o << decl << "[" << std::max<size_t>(v.size(), 1) << "] = {";
        if (v.empty()) o << "0.0";
        for (size_t i = 0; i < v.size(); ++i) o << lit(v[i]) << (i + 1 < v.size() ? ", " : "");
        o << "};\n";
    };
    const std::string ci = "__constant__ int ", cd = "__constant__ double ";
    o << "// by position: species, its T_mid, W and 1/W (0 where none sits); the NASA-7\n"
         "// rows, coefficient by coefficient, low range then high, so that the lanes of\n"
         "// a group read consecutive words\n";
    ints(ci + "PSPEC", pspec);
    std::vector<double> tm, pw(2 * npt, 0.0), th;
    for (int q = 0; q < npt; ++q) {
        const int k = pspec[q];
        tm.push_back(k >= 0 ? m.species[k].tmid : 1000.0);
        if (k >= 0) {
            pw[q] = m.species[k].W;
            pw[npt + q] = 1.0 / m.species[k].W;
        }
    }
    for (int c = 0; c < 19; ++c)
        for (int half = 0; half < 2; ++half)
            for (int q = 0; q < npt; ++q) {
                const int k = pspec[q];
                if (k < 0) {
                    th.push_back(0.0);
                    continue;
                }
                const double* a = half == 0 ? m.species[k].lo : m.species[k].hi;
                const double v[19] = {a[0], a[1], a[2], a[3], a[4], a[1] / 2, a[2] / 3, a[3] / 4, a[4] / 5,
                                      a[5], a[1] / 2, a[2] / 6, a[3] / 12, a[4] / 20, a[6] - a[0],
                                      a[1], 2 * a[2], 3 * a[3], 4 * a[4]};
                th.push_back(v[c]);
            }
    dbls(cd + "PTMID", tm);
    dbls(cd + "PW", pw);
    dbls(cd + "TH", th);
    o << "// species in position order: 1/W, original index\n";
    std::vector<double> iwm;
    for (int q = 0; q < ns; ++q) iwm.push_back(1.0 / m.species[ord[q]].W);
    dbls(cd + "IWM", iwm);
    ints(ci + "COLSPEC", ord);
    // per slot: words of reactant, then product species (position order, a byte
    // each, ns: none), then kind | irreversible << 3 | product form of K_c << 4 |
    // (dnu + 4) << 5 | reactant slots << 8 | product slots << 12 | row << 16
    std::vector<std::vector<int>> rs(nr), ps(nr);
    std::vector<int> row(nr, 0);
    std::vector<int> tb;                    // slots with a third body, in order
    std::vector<double> low, troe, plog;
    std::vector<int> plog_off(1, 0);
    for (int s = 0; s < nr; ++s) {
        const auto& r = m.reactions[order[s]];
        for (const auto& t : r.reac)
            for (int q = 0; q < t.nu; ++q) rs[s].push_back(inv[t.sp]);
        for (const auto& t : r.prod)
            for (int q = 0; q < t.nu; ++q) ps[s].push_back(inv[t.sp]);
        if (r.kind == RxnKind::Plog) {
            row[s] = (int)plog_off.size() - 1;
            for (const auto& x : r.plog) plog.insert(plog.end(), {x.lnp, x.lnA, x.b, x.EaR});
            plog_off.push_back((int)(plog.size() / 4));
        } else if (has_third_body(r.kind)) {
            row[s] = (int)tb.size();
            tb.push_back(s);
            low.insert(low.end(), {r.lnA0, r.b0, r.EaR0});
            const bool tr = r.kind == RxnKind::Troe;
            if (r.kind == RxnKind::Sri)
                troe.insert(troe.end(), {r.sri[0], -r.sri[1], 1.0 / r.sri[2], r.sri[1], std::log(r.sri[3]), r.sri[4],
                                         0.0, 0.0});
            else
                troe.insert(troe.end(), {tr ? 1.0 - r.alpha : 0.0, tr ? r.alpha : 0.0, tr ? 1.0 / r.T3 : 0.0,
                                         tr ? 1.0 / r.T1 : 0.0, tr && r.has_T2 ? r.T2 : 0.0,
                                         tr ? -(1.0 - r.alpha) / r.T3 : 0.0, tr ? -r.alpha / r.T1 : 0.0,
                                         tr && r.has_T2 ? 1.0 : 0.0});
        }
    }
    const int wr = (w.molr + 3) / 4, wp = (w.molp + 3) / 4;
    std::vector<int> packed((size_t)(wr + wp + 1) * nr);
    for (int s = 0; s < nr; ++s) {
        const auto& r = m.reactions[order[s]];
        for (int side = 0; side < 2; ++side) {
            const auto& v = side == 0 ? rs[s] : ps[s];
            const int nw = side == 0 ? wr : wp;
            for (int q = 0; q < nw; ++q) {
                unsigned x = 0;
                for (int b = 0; b < 4; ++b)
                    x |= (unsigned)(4 * q + b < (int)v.size() ? v[4 * q + b] : ns) << (8 * b);
                packed[(size_t)(side * wr + q) * nr + s] = (int)x;
            }
        }
        const bool pform = r.reversible && e.kc.product_form[order[s]];
        packed[(size_t)(wr + wp) * nr + s] =
            (int)((unsigned)r.kind | (r.reversible ? 0u : 8u) | (pform || !r.reversible ? 16u : 0u) |
                  ((unsigned)(r.dnu + 4) << 5) | ((unsigned)rs[s].size() << 8) | ((unsigned)ps[s].size() << 12) |
                  ((unsigned)row[s] << 16));
    }
    o << "// reactions in evaluation order (slot s): original index; packed words\n";
    ints(ci + "RX_ORIG", order);
    ints(ci + "RX_WORDS", packed);
    o << "// third-body and falloff slots, in order: low-pressure limit (ln A0 SI, b0, Ea0/R);\n"
         "// Troe: 1-alpha, alpha, 1/T***, 1/T*, T**, -(1-alpha)/T***, -alpha/T*, [T** given];\n"
         "// SRI: a, -b, 1/c, b, ln d, e; the collision partners of efficiency other than 1\n"
         "// and that efficiency less 1\n";
    auto columns = [&](const std::vector<double>& v, int n) {    // row by row -> column by column
        std::vector<double> c;
        for (int q = 0; q < n; ++q)
            for (int t = 0; t < w.ntb; ++t) c.push_back(v[(size_t)t * n + q]);
        return c;
    };
    dbls(cd + "RX_LOW", columns(low, 3));
    dbls(cd + "RX_TROE", columns(troe, 8));
    std::vector<int> tsp((size_t)w.maxp * w.ntb, ns);
    std::vector<double> tc((size_t)w.maxp * w.ntb, 0.0);
    for (int t = 0; t < w.ntb; ++t) {
        const auto& r = m.reactions[order[tb[t]]];
        const auto p = partners(r);
        for (size_t q = 0; q < p.size(); ++q) {
            tsp[q * w.ntb + t] = inv[p[q]];
            tc[q * w.ntb + t] = r.eff[p[q]] - 1.0;
        }
    }
    ints(ci + "TBP_SP", tsp);
    dbls(cd + "TBP_C", tc);
    o << "// PLOG tables: entries RX_PLOG_OFF[t] .. RX_PLOG_OFF[t+1] of (ln p, ln A SI, b, Ea/R)\n";
    ints(ci + "RX_PLOG_OFF", plog_off);
    dbls(cd + "RX_PLOG", plog);

    // Lists by position, 16 lanes side by side, each padded to the longest of
    // its 16.  A word: byte offset from the first reaction array | coefficient
    // << 24; padding points at an entry that stays zero, with coefficient 0.
    const int nrw = nr + 1, narr = std::max(5, w.molr + w.molp), zero = nr;
    auto net = [&](int s, int k) {
        int v = 0;
        for (int x : rs[s]) v -= x == k;
        for (int x : ps[s]) v += x == k;
        return v;
    };
    auto word = [](int idx, int nu) { return (int)((unsigned)idx * 8u | ((unsigned)nu << 24)); };
    // one list per position row, walked four words at a time and two such rows
    // a turn
    struct Lists {
        std::vector<int> len, data;
    };
    auto longest = [](const std::vector<std::vector<int>>& lanes) {
        size_t n = 0;
        for (const auto& v : lanes) n = std::max(n, v.size());
        return n;
    };
    auto add = [&](Lists& l, const std::vector<std::vector<int>>& lanes, int padding) {
        const size_t n = (longest(lanes) + 7) / 8 * 8;
        l.len.push_back((int)(n / 4));
        for (size_t t = 0; t < n; ++t)
            for (int i = 0; i < 16; ++i) l.data.push_back(t < lanes[i].size() ? lanes[i][t] : padding);
    };
    Lists wl, dl, dgl;
    for (int r = 0; r < w.r; ++r) {
        std::vector<std::vector<int>> lw(16), ld(16);
        for (int i = 0; i < 16; ++i) {
            const int k = 16 * r + i - 1;
            if (k < 0 || k >= na) continue;
            for (int s = 0; s < nr; ++s)
                if (const int v = net(s, k)) lw[i].push_back(word(s, v));
            for (int t = 0; t < w.ntb; ++t)
                if (const int v = net(tb[t], k)) ld[i].push_back(word(narr * nrw + t, v));
        }
        add(wl, lw, word(zero, 0));
        add(dl, ld, word(zero, 0));
    }
    // Jacobian rows, column by column, but a species' own column in a list of
    // its own (all its reactions are in it, a few of them in any other column,
    // and each column's lists are as long as the longest)
    std::vector<std::vector<std::vector<std::vector<int>>>> jlist(w.r);
    for (int r = 0; r < w.r; ++r) {
        std::vector<std::vector<int>> lg(16);
        for (int c = 0; c < ns; ++c) {
            std::vector<std::vector<int>> lj(16);
            for (int i = 0; i < 16; ++i) {
                const int k = 16 * r + i - 1;
                if (k < 0 || k >= na) continue;
                for (int s = 0; s < nr; ++s) {
                    const int v = net(s, k);
                    if (!v) continue;
                    for (size_t q = 0; q < rs[s].size(); ++q)
                        if (rs[s][q] == c) lj[i].push_back(word((int)q * nrw + s, v));
                    if (m.reactions[order[s]].reversible)
                        for (size_t q = 0; q < ps[s].size(); ++q)
                            if (ps[s][q] == c) lj[i].push_back(word((w.molr + (int)q) * nrw + s, v));
                }
                for (int t = 0; t < w.ntb; ++t) {
                    const int v = net(tb[t], k);
                    for (int q = 0; v && q < w.maxp; ++q)
                        if (tsp[(size_t)q * w.ntb + t] == c && tc[(size_t)q * w.ntb + t] != 0.0)
                            lj[i].push_back(word(narr * nrw + w.ntb + t * w.maxp + q, v));
                }
            }
            const int own = c + 1 - 16 * r;
            if (own >= 0 && own < 16 && c < na) lg[own].swap(lj[own]);
            jlist[r].push_back(lj);
        }
        add(dgl, lg, word(zero, 0));
    }
    // in groups of JGW columns of similar list length, walked side by side; the
    // groups of the columns of species some reaction changes come first
    const int jgw = 8;
    std::vector<int> grow, gcol, glen, jdata;
    int jgact = 0;
    for (int part = 0; part < 2; ++part) {
        for (int r = 0; r < w.r; ++r) {
            std::vector<int> cols;
            for (int c = part == 0 ? 0 : na; c < (part == 0 ? na : ns); ++c) cols.push_back(c);
            std::stable_sort(cols.begin(), cols.end(), [&](int a, int b) {
                return longest(jlist[r][a]) > longest(jlist[r][b]);
            });
            for (size_t g = 0; g < cols.size(); g += jgw) {
                const size_t n = (longest(jlist[r][cols[g]]) + 1) / 2 * 2;
                grow.push_back(r);
                glen.push_back((int)n);
                for (int q = 0; q < jgw; ++q) gcol.push_back(g + q < cols.size() ? cols[g + q] : -1);
                for (size_t t = 0; t < n; ++t)
                    for (int q = 0; q < jgw; ++q)
                        for (int i = 0; i < 16; ++i) {
                            const bool in = g + q < cols.size() && t < jlist[r][cols[g + q]][i].size();
                            jdata.push_back(in ? jlist[r][cols[g + q]][i][t] : word(zero, 0));
                        }
            }
        }
        if (part == 0) jgact = (int)grow.size();
    }
    // (the lists follow one another in the order the evaluation walks them; two
    // spare rows at the end, as words are loaded two rows ahead)
    std::vector<int> rl;
    for (const auto& q : {std::make_pair("W", &wl), std::make_pair("D", &dl), std::make_pair("DG", &dgl)}) {
        ints(std::string("constexpr int ") + q.first + "LEN", q.second->len);
        rl.insert(rl.end(), q.second->data.begin(), q.second->data.end());
    }
    rl.insert(rl.end(), 8 * 16, 0);
    o << "// by row: production rates (reaction slot, net coefficient); third-body part of a\n"
         "// Jacobian row (d q / d [M] of the slots that change the species); the species'\n"
         "// own column of it\n";
    // the words of a row that a lane takes lie together, so it reads four at once
    auto by_lane = [](const std::vector<int>& v, int lists) {
        std::vector<int> w(v.size());
        for (size_t k = 0; k < v.size(); ++k) {
            const size_t row = k / (16 * lists), q = k / 16 % lists, lane = k % 16;
            w[(row * 16 + lane) * lists + q] = v[k];
        }
        return w;
    };
    const std::string aligned = "__constant__ __attribute__((aligned(16))) int ";
    ints(aligned + "RL", by_lane(rl, 4));
    o << "// Jacobian rows, other columns: partials of the slots and third-body corrections,\n"
         "// in groups of columns\n"
      << "constexpr int JGW = " << jgw << ", JGACT = " << jgact << ", JGALL = " << grow.size() << ";\n";
    ints("constexpr int JGROW", grow);
    ints("constexpr int JGLEN", glen);
    ints("constexpr int JGCOL", gcol);
    jdata.insert(jdata.end(), 2 * jgw * 16, 0);
    ints(aligned + "JL", by_lane(jdata, jgw));
    o << "}  // namespace mech\n";
    return o.str();
}

// ---- the wave-cooperative adjoint: one matrix row per lane ----

RowLayout row_layout(const MechanismData& m)
{
    RowLayout w;
    const int ns = m.ns(), nr = m.nr(), n = ns + 1;
    if (n > 64) {
        w.G = 0;
        return w;
    }
    w.G = 16;
    while (w.G < n) w.G *= 2;
    w.maxt = 1;
    for (const auto& r : m.reactions) w.maxt = std::max<int>(w.maxt, (int)std::max(r.reac.size(), r.prod.size()));
    if (w.maxt > 3) {
        w.G = 0;
        return w;
    }
    for (const auto& r : m.reactions) {   // the packed reaction table's field widths
        for (const auto* side : {&r.reac, &r.prod})
            for (const auto& t : *side)
                if (t.nu > 3) w.G = 0;
        if (r.dnu < -4 || r.dnu > 3) w.G = 0;
    }
    int n_eff = 0, n_plog = 0;
    for (const auto& r : m.reactions) {
        if (r.kind == RxnKind::Plog) ++n_plog;
        else if (r.kind != RxnKind::Elementary) ++n_eff;
    }
    if (n_eff > 511 || n_plog > 511 || nr > 65535 || w.G == 0) {
        w.G = 0;
        return w;
    }
    w.nslot = 2 * w.maxt;
    w.pw = w.nslot + 2;
    w.jw = (ns + 1) % 2 ? ns + 1 : ns + 2;
    w.l_y = 0;
    w.l_c = w.l_y + n;
    w.l_g = w.l_c + ns;
    w.l_h = w.l_g + ns;
    w.l_q = w.l_h + ns;
    w.l_p = w.l_q + nr;
    w.l_j = w.l_p + nr * w.pw;
    w.l_t0 = w.l_j + ns * w.jw;
    w.l_w = w.l_t0 + ns;
    w.lds_cell = w.l_w + n;
    w.adj_lds_cell = 2 * w.lds_cell + 2 * n;
    return w;
}

std::string generate_row_source(const MechanismData& m, const RowLayout& w)
{
    Emitter e(m);
    std::ostringstream& o = e.o;
    const int ns = m.ns(), nr = m.nr();
    o << "// generated mechanism tables (wave-cooperative adjoint): " << m.name << " (" << ns << " species, " << nr
      << " reactions)\n"
      << "namespace mech {\n"
      << "constexpr int NS = " << ns << ";\n"
      << "constexpr int NR = " << nr << ";\n"
      << "constexpr int N = NS + 1;\n"
      << "constexpr int G = " << w.G << ";            // lanes per cell\n"
      << "constexpr int MAXT = " << w.maxt << ";         // most terms on a reaction side\n"
      << "constexpr int NSLOT = " << w.nslot << ", PW = " << w.pw << ", JW = " << w.jw << ";\n"
      << "constexpr int L_Y = " << w.l_y << ", L_C = " << w.l_c << ", L_G = " << w.l_g << ", L_H = " << w.l_h
      << ", L_Q = " << w.l_q << ", L_P = " << w.l_p << ", L_J = " << w.l_j << ", L_T0 = " << w.l_t0
      << ", L_W = " << w.l_w << ";\n"
      << "constexpr int LDS_CELL = " << w.lds_cell << ";  // doubles of LDS scratch per cell\n"
      << "constexpr int ADJ_LDS_CELL = " << w.adj_lds_cell << ";  // per cell in the adjoint\n"
      << "constexpr double RU = " << lit(kRu) << ";\n"
      << "constexpr double LN_PATM_R = " << lit(std::log(kPatm / kRu)) << ";\n"
      << "constexpr double LN10 = " << lit(std::log(10.0)) << ";\n";
    e.thermo_table();
    o << "__constant__ double TMID[NS] = {";
    for (int k = 0; k < ns; ++k) o << lit(m.species[k].tmid) << (k + 1 < ns ? ", " : "};\n");
    // reactions in evaluation order: grouped by kind so a round of lanes mostly
    // takes one branch
    std::vector<int> order;
    for (int kind = 0; kind < 6; ++kind)
        for (int j = 0; j < nr; ++j)
            if ((int)m.reactions[j].kind == kind) order.push_back(j);
    std::vector<int> slot_of(nr);
    for (int s = 0; s < nr; ++s) slot_of[order[s]] = s;
    // per slot: its EFF row (third body and falloff) or its PLOG table (PLOG)
    std::vector<int> effrow(nr, -1);
    int neff = 0, nplog = 0;
    for (int s = 0; s < nr; ++s) {
        const RxnKind k = m.reactions[order[s]].kind;
        if (k == RxnKind::Plog) effrow[s] = nplog++;
        else if (k != RxnKind::Elementary) effrow[s] = neff++;
    }
    auto ints = [&](const char* name, const std::vector<int>& v) {
        o << "__constant__ int " << name << "[" << std::max<size_t>(v.size(), 1) << "] = {";
        if (v.empty()) o << "0";
        for (size_t i = 0; i < v.size(); ++i) o << v[i] << (i + 1 < v.size() ? ", " : "");
        o << "};\n";
    };
    auto dbls = [&](const char* name, const std::vector<double>& v) {
        o << "__constant__ double " << name << "[" << std::max<size_t>(v.size(), 1) << "] = {";
        if (v.empty()) o << "0.0";
        for (size_t i = 0; i < v.size(); ++i) o << lit(v[i]) << (i + 1 < v.size() ? ", " : "");
        o << "};\n";
    };
    // per slot: original index; species of the MAXT reactant then MAXT product
    // slots (-1: unused)
    std::vector<int> orig, sp;
    std::vector<double> low, troe, eff, plog;
    std::vector<int> plog_off(1, 0);
    for (int s = 0; s < nr; ++s) {
        const auto& r = m.reactions[order[s]];
        orig.push_back(order[s]);
        for (int t = 0; t < w.maxt; ++t) sp.push_back(t < (int)r.reac.size() ? r.reac[t].sp : -1);
        for (int t = 0; t < w.maxt; ++t) sp.push_back(t < (int)r.prod.size() ? r.prod[t].sp : -1);
        low.insert(low.end(), {r.lnA0, r.b0, r.EaR0});
        const bool tr = r.kind == RxnKind::Troe;
        if (r.kind == RxnKind::Sri)
            troe.insert(troe.end(), {r.sri[0], -r.sri[1], 1.0 / r.sri[2], r.sri[1], std::log(r.sri[3]), r.sri[4],
                                     0.0, 0.0});
        else
            troe.insert(troe.end(), {tr ? 1.0 - r.alpha : 0.0, tr ? r.alpha : 0.0, tr ? 1.0 / r.T3 : 0.0,
                                     tr ? 1.0 / r.T1 : 0.0, tr && r.has_T2 ? r.T2 : 0.0,
                                     tr ? -(1.0 - r.alpha) / r.T3 : 0.0, tr ? -r.alpha / r.T1 : 0.0,
                                     tr && r.has_T2 ? 1.0 : 0.0});
        if (r.kind == RxnKind::Plog) {
            for (const auto& e : r.plog) plog.insert(plog.end(), {e.lnp, e.lnA, e.b, e.EaR});
            plog_off.push_back((int)(plog.size() / 4));
        } else if (effrow[s] >= 0) {
            for (int k = 0; k < ns; ++k) eff.push_back(r.eff[k]);
        }
    }
    // packed per slot, for one load per reaction round: species slots (8 bits
    // each: species index + 1 in the low 6 bits, coefficient in the top 2;
    // 0 = unused) in two words, then kind | irreversible << 3 | (dnu + 4) << 4 |
    // (EFF row or PLOG table + 1) << 7 | orig << 16
    {
        std::vector<int> pack;
        for (int s = 0; s < nr; ++s) {
            const auto& r = m.reactions[order[s]];
            unsigned long long slots = 0;
            for (int t = 0; t < 2 * w.maxt; ++t) {
                const bool isr = t < w.maxt;
                const auto& side = isr ? r.reac : r.prod;
                const int q = isr ? t : t - w.maxt;
                unsigned v = 0;
                if (q < (int)side.size()) v = (unsigned)(side[q].sp + 1) | ((unsigned)side[q].nu << 6);
                slots |= (unsigned long long)v << (8 * t);
            }
            pack.push_back((int)(unsigned)(slots & 0xffffffffull));
            pack.push_back((int)(unsigned)(slots >> 32));
            pack.push_back((int)((unsigned)r.kind | ((r.reversible ? 0u : 1u) << 3) | ((unsigned)(r.dnu + 4) << 4) |
                                 ((unsigned)(effrow[s] + 1) << 7) | ((unsigned)order[s] << 16)));
        }
        o << "// per slot: species slots (two words, 8 bits each: index + 1 | nu << 6), then\n"
             "// kind | irreversible << 3 | (dnu + 4) << 4 | (EFF row or PLOG table + 1) << 7 |\n"
             "// original index << 16\n";
        ints("RX_PACK", pack);
    }
    o << "// reactions in evaluation order (slot s): original index (kind, species\n"
         "// slots and coefficients are in RX_PACK)\n";
    ints("RX_ORIG", orig);
    o << "// low-pressure limit (ln A0 SI, b0, Ea0/R); Troe: 1-alpha, alpha, 1/T***,\n"
         "// 1/T*, T**, -(1-alpha)/T***, -alpha/T*, [T** given]; SRI: a, -b, 1/c, b, ln d, e\n";
    dbls("RX_LOW", low);
    dbls("RX_TROE", troe);
    {
        bool sri = false, irrev = false;
        for (const auto& r : m.reactions) {
            sri = sri || r.kind == RxnKind::Sri;
            irrev = irrev || !r.reversible;
        }
        o << "// reaction forms present (the kernels leave out the code of the absent ones)\n"
             "constexpr bool HAS_PLOG = " << (nplog > 0 ? "true" : "false") << ";\n"
             "constexpr bool HAS_SRI = " << (sri ? "true" : "false") << ";\n"
             "constexpr bool HAS_IRREV = " << (irrev ? "true" : "false") << ";\n";
    }
    o << "// PLOG tables: entries RX_PLOG_OFF[t] .. RX_PLOG_OFF[t+1] of (ln p, ln A SI, b, Ea/R)\n";
    ints("RX_PLOG_OFF", plog_off);
    dbls("RX_PLOG", plog);
    o << "// third-body efficiencies, one dense row per non-elementary reaction\n";
    dbls("EFF", eff);
    // species -> reactions that change it (slot, net coefficient)
    std::vector<int> off(1, 0), srx, snu;
    for (int k = 0; k < ns; ++k) {
        for (int s = 0; s < nr; ++s) {
            const auto& r = m.reactions[order[s]];
            int v = 0;
            for (auto& t : r.reac) if (t.sp == k) v -= t.nu;
            for (auto& t : r.prod) if (t.sp == k) v += t.nu;
            if (v) {
                srx.push_back(s);
                snu.push_back(v);
            }
        }
        while ((srx.size() - off.back()) % 4) {   // padded to a multiple of 4 (coefficient 0)
            srx.push_back(0);
            snu.push_back(0);
        }
        off.push_back((int)srx.size());
    }
    o << "// species k: the reactions that change it, SP_RX[SP_OFF[k] .. SP_OFF[k+1]),\n"
         "// with net coefficients SP_NU (padded to a multiple of 4 by coefficient 0)\n";
    ints("SP_OFF", off);
    ints("SP_RX", srx);
    ints("SP_NU", snu);
    // the same entries packed for the Jacobian rows, so one round of loads gives
    // everything an entry needs: slot | (net coefficient & 255) << 16, then the
    // species of the reaction's slots 0-3 and 4-5 as bytes (index + 1, 0 unused)
    {
        std::vector<int> jp;
        for (size_t e = 0; e < srx.size(); ++e) {
            const int slot = srx[e];
            jp.push_back((int)((unsigned)slot | (((unsigned)snu[e] & 255u) << 16)));
            unsigned b[2] = {0u, 0u};
            for (int t = 0; t < w.nslot; ++t) {
                const int spc = sp[slot * w.nslot + t];
                b[t / 4] |= (unsigned)(spc + 1) << (8 * (t % 4));
            }
            jp.push_back((int)b[0]);
            jp.push_back((int)b[1]);
        }
        o << "// per SP entry: slot | (net coefficient & 255) << 16, slot species 0-3, 4-5 (bytes, index + 1)\n";
        ints("SP_JPACK", jp);
    }
    // third-body and falloff reactions t (EFF row t): their slot, and the net
    // coefficient of every species in them (the dense third-body part of the
    // Jacobian rows)
    std::vector<int> tbslot;
    std::vector<double> nutb;
    for (int s = 0; s < nr; ++s)
        if (effrow[s] >= 0 && m.reactions[order[s]].kind != RxnKind::Plog) tbslot.push_back(s);
    for (int k = 0; k < ns; ++k)
        for (int s : tbslot) {
            const auto& r = m.reactions[order[s]];
            int v = 0;
            for (auto& t : r.reac) if (t.sp == k) v -= t.nu;
            for (auto& t : r.prod) if (t.sp == k) v += t.nu;
            nutb.push_back((double)v);
        }
    o << "constexpr int NTB = " << tbslot.size() << ";\n"
         "static_assert(NTB == 0 || sizeof(EFF) == sizeof(double) * NTB * NS, \"one EFF row per third-body "
         "reaction\");\n"
         "// third-body or falloff reaction t: its slot (EFF row t); the net coefficient of\n"
         "// species k in it as a 4-bit field (coefficient + 8), eight per word:\n"
         "// NU_TB4[k * NTBW + t / 8] >> (4 (t % 8))\n";
    ints("TB_SLOT", tbslot);
    {
        const int ntb = (int)tbslot.size(), ntbw = std::max(1, (ntb + 7) / 8);
        std::vector<int> packed((size_t)ns * ntbw, 0);
        for (int k = 0; k < ns; ++k)
            for (int t = 0; t < ntb; ++t) {
                const int v = (int)nutb[(size_t)k * ntb + t];
                packed[(size_t)k * ntbw + t / 8] |= (int)((unsigned)(v + 8) << (4 * (t % 8)));
            }
        o << "constexpr int NTBW = " << ntbw << ";\n";
        ints("NU_TB4", packed);
    }
    o << "}  // namespace mech\n";
    return o.str();
}

}  // namespace chemmi
