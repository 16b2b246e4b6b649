// wide.hip -- the chemistry step for mechanisms whose per-cell matrices do not
// fit the registers of one lane (CDNA4, gfx950).
//
// G = 16 lanes, one DPP row, cooperate on one cell, so a 64-lane wave holds
// four cells.  The components of the state are taken in the elimination order
// T, then the species some reaction changes (NACT positions), then the
// species no reaction changes.  Lane i owns the positions r * 16 + i for
// r < R = ceil(NACT / 16): their components of every state-sized vector, and
// their rows of the step matrix and of its LU factors, all in registers.
//
// Why 16 lanes and R rows a lane, not one row a lane: a broadcast from a lane
// of the group is then one in-row DPP move a register (row_newbcast), with no
// LDS round trip and no scalar register; the pivot search and the mixture
// sums are four DPP steps; and the work that every lane repeats (T's powers,
// the controller, the pivot's reciprocal) serves four cells a wave.  With a
// lane a row (64 lanes a cell at 33 unknowns, 32 at 17) the same step took
// 18.2 k vector instructions per cell and 68 us at 17 unknowns.
//
// A species no reaction changes has a zero source term and a zero row in the
// Jacobian, so all its stage vectors are exactly zero and its column of the
// step matrix never meets anything but zeros: the forward step is the
// NACT x NACT system.  Such species enter the mixture sums and the third-body
// concentrations.
//
// Per source-term evaluation:
//   - species thermo (NASA-7) and equilibrium factors e^{+-G} in the lanes of
//     the species' positions;
//   - mixture sums (sum Y/W, c_p, heat release) as DPP butterflies, every lane
//     of the group ending with the same bits;
//   - reactions 16 at a time (lane i: slot q * 16 + i), those with third-body,
//     falloff or PLOG terms first, so that only the leading rounds run that code;
//   - production rates and Jacobian rows gathered by each lane from the cell's LDS through per-position lists padded to the
//     longest of the 16 lanes, so every loop has a compile-time length and
//     the sums have a fixed order (reproducible results).
//
// The equations, the RODAS4 tableau and the controller are those of the
// one-cell-per-lane integrator (the species/energy source of eqs. (20)-(21)
// at constant pressure over one flow step).

namespace chemw {

using chem::RA;
using chem::RC;
using chem::Rodas4;
using chem::StepArgs;
using chem::finite;
constexpr int N = mech::N, NS = mech::NS, NR = mech::NR, NA = mech::NA, NI = mech::NI;
constexpr int NACT = mech::NACT, R = mech::R, RI = mech::RI, NPT = mech::NPT;
constexpr int G = 16;
constexpr int SP = NS + 1;           // a species array in LDS, and a last entry of neutral elements
constexpr int NRW = NR + 1;          // a reaction array in LDS, and a last entry that stays zero
constexpr int MOLR = mech::MOLR, MOLP = mech::MOLP;
constexpr int MOLM = MOLR > MOLP ? MOLR : MOLP;
constexpr int WR = (MOLR + 3) / 4, WP = (MOLP + 3) / 4, NWORDS = WR + WP + 1;
constexpr int ROUNDS = (NR + G - 1) / G;
constexpr int NTB = mech::NTB, MAXP = mech::MAXP;
static_assert(R * 16 >= NACT && RI * 16 >= NI + 1, "positions");

// ---- LDS: the workgroup's tables, then one scratch per cell ----
// The tables that an evaluation reads at every reaction and species sit in
// LDS, one copy for the workgroup's waves: from global memory each read cost
// an L2 latency in the evaluation's chain (the vector L1 does not hold them
// all; 32 species: 12.2 k cycles for the reactions of an evaluation, 4.7 k for
// the thermo, one wave per SIMD).
//   doubles: ln A, b, Ea/R by slot; NASA-7 rows by position; low-pressure
//   limits, Troe/SRI constants and partner efficiencies of the third-body
//   slots; ints: packed words by slot, partner species
constexpr int T_PAR = 0;
constexpr int T_TH = 3 * NR;
constexpr int T_LOW = T_TH + 38 * NPT;
constexpr int T_TROE = T_LOW + 3 * NTB;
constexpr int T_TBC = T_TROE + 8 * NTB;
constexpr int T_INT = T_TBC + MAXP * NTB;                 // in doubles
constexpr int I_WORDS = 0, I_TBSP = NWORDS * NR, N_INT = NWORDS * NR + MAXP * NTB;
constexpr int TAB_DOUBLES = T_INT + (N_INT + 1) / 2;
// per cell: concentrations, e^{G}, e^{-G}, H/RT, then G itself where some
// reaction needs it, then the reaction arrays
constexpr int L_C = 0, L_GP = SP, L_GM = 2 * SP, L_H = 3 * SP;
constexpr int L_G = 4 * SP;
constexpr int L_A = (mech::HAS_LNKC ? 5 : 4) * SP;
constexpr int NARR = MOLR + MOLP > 5 ? MOLR + MOLP : 5;
constexpr int L_X = L_A + NARR * NRW;        // third-body terms: NTB, then NTB * MAXP partner corrections

__device__ __forceinline__ int gl() { return (int)(threadIdx.x & 15u); }
__device__ __forceinline__ int gbase() { return (int)(threadIdx.x & 48u); }

// the lane index behind an opaque zero: compares against it (i == k for every
// k of an unrolled loop) and table words loaded at it are made where used
// instead of being hoisted out of the substep loop as dozens of live masks and
// hundreds of live words
__device__ __forceinline__ int gl_local() { return gl() + mech::opaque_zero(); }

template <int K>
struct Int {
    static constexpr int v = K;
};

// f(Int<B>{}), ..., f(Int<E - 1>{}): a loop whose index is a constant in the
// body, for bounds and list lengths that depend on it
template <int B, int E, class Fn>
__device__ __forceinline__ void static_for(Fn&& f)
{
    if constexpr (B < E) {
        f(Int<B>{});
        static_for<B + 1, E>(f);
    }
}

template <int CTRL>
__device__ __forceinline__ double dpp(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// value of x in lane k of this group (k a compile-time constant after unrolling)
__device__ __forceinline__ double bc(double x, int k)
{
    switch (k & 15) {
    case 0: return dpp<0x150>(x);
    case 1: return dpp<0x151>(x);
    case 2: return dpp<0x152>(x);
    case 3: return dpp<0x153>(x);
    case 4: return dpp<0x154>(x);
    case 5: return dpp<0x155>(x);
    case 6: return dpp<0x156>(x);
    case 7: return dpp<0x157>(x);
    case 8: return dpp<0x158>(x);
    case 9: return dpp<0x159>(x);
    case 10: return dpp<0x15A>(x);
    case 11: return dpp<0x15B>(x);
    case 12: return dpp<0x15C>(x);
    case 13: return dpp<0x15D>(x);
    case 14: return dpp<0x15E>(x);
    default: return dpp<0x15F>(x);
    }
}

// value of x in lane `src` of this group; src may differ per lane
__device__ __forceinline__ double gather(double x, int src) { return __shfl(x, gbase() + src, 64); }

// Group reductions: a butterfly over the DPP patterns xor 1, xor 2,
// mirror-in-8 and mirror-in-16; each step adds a lane's value to its
// partner's and the partner adds the same two numbers, so every lane of the
// group ends with the same bits.
template <class Op>
__device__ __forceinline__ double greduce(double x, Op op)
{
    x = op(x, dpp<0xB1>(x));    // quad_perm [1, 0, 3, 2]
    x = op(x, dpp<0x4E>(x));    // quad_perm [2, 3, 0, 1]
    x = op(x, dpp<0x141>(x));   // row_half_mirror
    return op(x, dpp<0x140>(x));   // row_mirror
}
__device__ __forceinline__ double gsum(double x)
{
    return greduce(x, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double gmax(double x)
{
    return greduce(x, [](double a, double b) { return fmax(a, b); });
}

// true in every lane of the group if `bad` holds in any lane of it
__device__ __forceinline__ bool gany(bool bad)
{
    return ((__ballot(bad) >> gbase()) & 0xffffull) != 0ull;
}

// Order between the LDS accesses of one wave: its LDS instructions execute in
// program order, so only the compiler has to keep it.
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void load_tables(double* __restrict__ tab, const double* __restrict__ par)
{
    int* const ti = (int*)(tab + T_INT);
    const int t0 = (int)threadIdx.x, nt = (int)blockDim.x;
    for (int j = t0; j < NR; j += nt) {
        const int o = mech::RX_ORIG[j];
#pragma unroll
        for (int q = 0; q < 3; ++q) tab[T_PAR + q * NR + j] = par[q * NR + o];
    }
    for (int j = t0; j < 38 * NPT; j += nt) tab[T_TH + j] = mech::TH[j];
    for (int j = t0; j < 3 * NTB; j += nt) tab[T_LOW + j] = mech::RX_LOW[j];
    for (int j = t0; j < 8 * NTB; j += nt) tab[T_TROE + j] = mech::RX_TROE[j];
    for (int j = t0; j < MAXP * NTB; j += nt) {
        tab[T_TBC + j] = mech::TBP_C[j];
        ti[I_TBSP + j] = mech::TBP_SP[j];
    }
    for (int j = t0; j < NWORDS * NR; j += nt) ti[I_WORDS + j] = mech::RX_WORDS[j];
    __syncthreads();
}

// the temperature-dependent scalars of one evaluation, the same in every lane
struct Mix {
    double T, lnT, iT, lnPRT, ctot, rtp, prt;
    double p;
};

// One reaction's rate and derivatives.  q: rate of progress; the others as far
// as the evaluation needs them: kf, kr the (third-body scaled) rate constants
// of the two sides; dqT = d q / d T at fixed C; dM the coefficient of the
// third-body efficiencies in d q / d C; s = sum_m d q / d C_m C_m; qA = d q /
// d ln A of the main rate; dH = sum nu H/RT.
struct Rate {
    double q, kf, kr, dqT, dM, s, qA, dH;
};

// What a lane reads for its reaction, in two dependent LDS rounds: the table
// entries, and then the species' values that they name.  Each round is issued
// as a whole, and the next reaction's entries are read during this one's
// arithmetic; left to the compiler, loads and uses alternated, a wait apiece.
// A wave here is bound by such latencies, not by issue (vector instructions
// issued in 45 % of the cycles, 40 % in waits): with the same grouping of the
// list and thermo loads and the falloff terms as one block, a substep of a lone
// wave went from 84,800 to 64,200 cycles (16 species), and the 1M-cell field of
// 32 species from 27.0 to 21.2 ms.
struct Entry {
    double lnA, b, Ea;
    int w[NWORDS];

    __device__ __forceinline__ Entry(const double* __restrict__ tab, int j)
    {
        const int* const words = (const int*)(tab + T_INT) + I_WORDS;
        const int k = j < NR ? j : NR - 1;
        lnA = tab[T_PAR + k];
        b = tab[T_PAR + NR + k];
        Ea = tab[T_PAR + 2 * NR + k];
#pragma unroll
        for (int q = 0; q < NWORDS; ++q) w[q] = words[q * NR + k];
    }
};

template <bool DERIV>
struct Slots {
    int ra[MOLR], pa[MOLP];
    double cr[MOLR], cp[MOLP], gr[MOLR], gp[MOLP];   // C, e^{G} and e^{-G}
    double hr[DERIV ? MOLR : 1], hp[DERIV ? MOLP : 1];

    __device__ __forceinline__ Slots(const Entry& e, const double* __restrict__ L)
    {
#pragma unroll
        for (int s = 0; s < MOLR; ++s) {
            ra[s] = (e.w[s / 4] >> (8 * (s % 4))) & 255;
            cr[s] = L[L_C + ra[s]];
            gr[s] = L[L_GP + ra[s]];
            if (DERIV) hr[s] = L[L_H + ra[s]];
        }
#pragma unroll
        for (int s = 0; s < MOLP; ++s) {
            pa[s] = (e.w[WR + s / 4] >> (8 * (s % 4))) & 255;
            cp[s] = L[L_C + pa[s]];
            gp[s] = L[L_GM + pa[s]];
            if (DERIV) hp[s] = L[L_H + pa[s]];
        }
    }
};

// FULL: the round may hold slots other than elementary ones.
// DERIV: derivatives are wanted.
template <bool FULL, bool DERIV>
__device__ __forceinline__ void reaction(const Entry& en, const Slots<DERIV>& sl, const double* __restrict__ tab,
                                         const double* __restrict__ L, const Mix& x, Rate& o)
{
    const double lnA = en.lnA, pb = en.b, pe = en.Ea;
    const int misc = en.w[NWORDS - 1];
    double pf = sl.cr[0], pr = sl.cp[0];
#pragma unroll
    for (int s = 1; s < MOLR; ++s) pf = pf * sl.cr[s];
#pragma unroll
    for (int s = 1; s < MOLP; ++s) pr = pr * sl.cp[s];
    // 1/K_c = prod_reac e^{G} prod_prod e^{-G} (RT/P_atm)^dnu, the factors
    // multiplied reactant, product, reactant, ... as the range check took them
    double ikc = sl.gr[0] * sl.gp[0];
#pragma unroll
    for (int s = 1; s < MOLM; ++s) {
        if (s < MOLR) ikc = ikc * sl.gr[s < MOLR ? s : 0];
        if (s < MOLP) ikc = ikc * sl.gp[s < MOLP ? s : 0];
    }
    const int dnu = ((misc >> 5) & 7) - 4;
#pragma unroll
    for (int q = 1; q <= mech::MAXDNU; ++q) {
        const double f = dnu > 0 ? x.rtp : x.prt;
        ikc = (dnu >= q || dnu <= -q) ? ikc * f : ikc;
    }
    // (K_c out of the range of the factors: by its logarithm)
    const bool by_log = mech::HAS_LNKC && !((misc >> 4) & 1);
    double lnKc = 0.0;
    if (by_log) {
        lnKc = (double)dnu * x.lnPRT;
#pragma unroll
        for (int s = 0; s < MOLR; ++s) lnKc = lnKc - L[L_G + sl.ra[s]];
#pragma unroll
        for (int s = 0; s < MOLP; ++s) lnKc = lnKc + L[L_G + sl.pa[s]];
        ikc = chem_math::exp_poly(-lnKc);
    }
    if (mech::HAS_IRREV && ((misc >> 3) & 1)) ikc = 0.0;
    double lnk = x.lnT * pb;
    lnk = fma(-x.iT, pe, lnk);
    lnk = lnk + lnA;
    const int kind = FULL ? misc & 7 : 0;
    double eb = pb, ee = pe;
    if (FULL && mech::HAS_PLOG && kind == 5) {
        // the Arrhenius set at this pressure: linear in ln p between the
        // tabulated pressures, the end sets outside them
        const double lnp = chem_math::ln(x.p);
        const int t = (misc >> 16) & 0xffff;
        const int e0 = mech::RX_PLOG_OFF[t], e1 = mech::RX_PLOG_OFF[t + 1] - 1;
        const double* E = mech::RX_PLOG;
        int e = e0;
        double v = 0.0;
        if (lnp >= E[4 * e1]) {
            e = e1;
        } else if (lnp > E[4 * e0]) {
            while (e + 1 < e1 && lnp >= E[4 * (e + 1)]) ++e;
            v = (lnp - E[4 * e]) / (E[4 * (e + 1)] - E[4 * e]);
        }
        const int e2 = e < e1 ? e + 1 : e;
        const double pla = fma(v, E[4 * e2 + 1] - E[4 * e + 1], E[4 * e + 1]);
        const double plb = fma(v, E[4 * e2 + 2] - E[4 * e + 2], E[4 * e + 2]);
        const double ple = fma(v, E[4 * e2 + 3] - E[4 * e + 3], E[4 * e + 3]);
        lnk = lnk + (x.lnT * plb - x.iT * ple + pla);
        eb += plb;
        ee += ple;
    }
    double kf, fac = 1.0, Mc = 0.0, dkdM = 0.0, qAf = 1.0, dlnkf = 0.0;
    if (DERIV) dlnkf = (eb + ee * x.iT) * x.iT;
    const bool third = FULL && NTB > 0 && kind >= 1 && kind <= 4, fall = third && kind >= 2;
    if (FULL && NTB > 0) {
        const int t = third ? (misc >> 16) & 0xffff : 0;
        Mc = x.ctot;
        constexpr int TB = MAXP < 4 ? (MAXP > 0 ? MAXP : 1) : 4;      // partners read together
#pragma unroll 1
        for (int q0 = 0; q0 < MAXP; q0 += TB) {
            double tc[TB], tl[TB];
#pragma unroll
            for (int q = 0; q < TB; ++q) {
                const int k = q0 + q < MAXP ? q0 + q : MAXP - 1;
                tc[q] = tab[T_TBC + k * NTB + t];
                tl[q] = L[L_C + ((const int*)(tab + T_INT))[I_TBSP + k * NTB + t]];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < TB; ++q)
                if (q0 + q < MAXP) Mc = fma(tl[q], tc[q], Mc);
        }
        if (kind == 1) fac = Mc;
    }
    if (FULL && NTB > 0 && __any(fall)) {
        // Falloff, in all lanes of a wave that has some, kept in those that are:
        // as one block the exponentials and logarithms that do not depend on one
        // another (k_inf, P_r, the terms of F_cent) overlap; branch by branch
        // they followed one another.
        // P_r = k0 [M] / k_inf, one exponential for the ratio
        const int t = third ? (misc >> 16) & 0xffff : 0;
        const double* lo = tab + T_LOW + t;
        const double* tr = tab + T_TROE + t;
        double lw[3], tw[8];
#pragma unroll
        for (int k = 0; k < 3; ++k) lw[k] = lo[k * NTB];
#pragma unroll
        for (int k = 0; k < 8; ++k) tw[k] = tr[k * NTB];
        __builtin_amdgcn_sched_barrier(0);
        kf = chem_math::exp_poly(lnk);
        const double lnr0 = lw[0] + lw[1] * x.lnT - lw[2] * x.iT - lnk;
        const double r0 = chem_math::exp_poly(lnr0);
        const double Pr = r0 * Mc;
        const bool floored = !(Pr >= 1e-300);
        const double lgPr = chem_math::lg(Pr);
        const double logPr = floored ? -300.0 : lgPr;
        const double ipr1 = chem_math::recip(1.0 + Pr);
        double Fb = 1.0, dF_dPr = 0.0, dlnF_T = 0.0;
        if (mech::HAS_TROE) {
            const bool troe = kind == 3;
            const double e3 = chem_math::exp_neg(-x.T * tw[2]);
            const double e1 = chem_math::exp_neg(-x.T * tw[3]);
            const double e2 = chem_math::exp_neg(-tw[4] * x.iT);
            const double Fc3 = tw[0] * e3 + tw[1] * e1;
            const double dFc3 = tw[5] * e3 + tw[6] * e1;
            const bool four = tw[7] != 0.0;
            const double Fc = four ? Fc3 + e2 : Fc3;
            const double dFc = four ? dFc3 + tw[4] * x.iT * x.iT * e2 : dFc3;
            const double logFc = chem_math::lg(Fc);
            const double tc = -0.4 - 0.67 * logFc;
            const double tn = 0.75 - 1.27 * logFc;
            const double tu = logPr + tc;
            const double itd = chem_math::recip(tn - 0.14 * tu);
            const double tx = tu * itd;
            const double iop = chem_math::recip(1.0 + tx * tx);
            const double logF = logFc * iop;
            const double Ft = chem_math::exp_neg(mech::LN10 * logF);
            Fb = troe ? Ft : Fb;
            if (DERIV) {
                const double tg = -logFc * 2.0 * tx * (iop * iop);
                const double d = tg * tn * (itd * itd);
                dF_dPr = troe && !floored ? d : dF_dPr;
                const double dF_dFc = iop + tg * (-0.67 * tn + 1.27 * tu) * (itd * itd);
                const double dT = mech::LN10 * dF_dFc * (dFc / (Fc * mech::LN10));
                dlnF_T = troe ? dT : dlnF_T;
            }
        }
        if (mech::HAS_SRI && kind == 4) {
            // SRI: F = d [a exp(-b/T) + exp(-T/c)]^X T^e, X = 1 / (1 + log10(P_r)^2);
            // row: a, -b, 1/c, b, ln d, e
            const double sea = tw[0] * chem_math::exp_neg(tw[1] * x.iT);
            const double sec = chem_math::exp_neg(-x.T * tw[2]);
            const double sY = sea + sec;
            const double lnsY = chem_math::ln<true>(sY);
            const double sX = chem_math::recip(1.0 + logPr * logPr);
            Fb = chem_math::exp_poly(sX * lnsY + tw[5] * x.lnT + tw[4]);
            if (DERIV) {
                if (!floored) dF_dPr = lnsY * (-2.0 / mech::LN10) * logPr * sX * sX;
                dlnF_T = sX * (sea * tw[3] * x.iT * x.iT - sec * tw[2]) / sY + tw[5] * x.iT;
            }
        }
        if (DERIV) {
            const double dlnk0 = (lw[1] + lw[2] * x.iT) * x.iT;
            const double dl = dlnkf + (ipr1 + dF_dPr) * (dlnk0 - dlnkf) + dlnF_T;
            dlnkf = fall ? dl : dlnkf;
            dkdM = kf * r0 * Fb * (ipr1 * ipr1 + dF_dPr * ipr1);
            qAf = fall ? Pr * ipr1 - dF_dPr : 1.0;
        }
        const double kl = kf * Pr * ipr1 * Fb;
        kf = fall ? kl : kf;
    } else {
        kf = chem_math::exp_poly(lnk);
    }
    const double net = fma(-ikc, pr, pf);
    double kfn = kf * net, kr = kf * ikc;
    if (by_log && !fall) {
        // 1/K_c may be beyond the largest double, and k_f below the smallest,
        // where their product, the reverse rate constant, is an ordinary number
        kr = chem_math::exp_poly(lnk - lnKc);
        kfn = kf * pf - kr * pr;
    }
    o.q = FULL ? fac * kfn : kfn;
    if (DERIV) {
        o.kf = FULL ? fac * kf : kf;
        o.kr = FULL ? fac * kr : kr;
        const double fwd = o.kf * pf, rev = o.kr * pr;
        double dH = 0.0;
#pragma unroll
        for (int s = 0; s < MOLP; ++s) dH = dH + sl.hp[s];
#pragma unroll
        for (int s = 0; s < MOLR; ++s) dH = dH - sl.hr[s];
        o.dH = dH;
        const double dlnKc = (dH - (double)dnu) * x.iT;
        o.dqT = dlnkf * fwd - (dlnkf - dlnKc) * rev;
        o.s = (double)((misc >> 8) & 15) * fwd - (double)((misc >> 12) & 15) * rev;
        o.dM = 0.0;
        o.qA = o.q;
        if (FULL && NTB > 0 && kind >= 1 && kind <= 4) {
            o.dM = kind == 1 ? kfn : dkdM * net;
            o.s = o.s + Mc * o.dM;
            if (kind >= 2) o.qA = o.q * qAf;
        }
    }
}

// product of the concentrations of a side's slots but s (times c)
template <int MOL>
__device__ __forceinline__ double others(const double* __restrict__ L, const int (&a)[MOL], int s, double c)
{
#pragma unroll
    for (int t = 0; t < MOL; ++t)
        if (t != s) c = c * L[L_C + a[t]];
    return c;
}

// Species thermo, mixture sums and the species arrays in LDS: the part of an
// evaluation before the reactions.  y: the lane's components; ywi: Y/W of its
// species that no reaction changes.
template <bool DERIV>
struct Thermo {
    double cpR[R], HRT[R], yw[R], dcpR[DERIV ? R : 1];
    double cpi[RI];
    double rho, irho, Wbar, sig, cpm, dcpm;
};

template <bool DERIV>
__device__ __forceinline__ void thermo(const double* __restrict__ tab, double p, double ip, const double (&y)[R], const double (&ywi)[RI],
                                       double* __restrict__ L, Mix& x, Thermo<DERIV>& th)
{
    const int i = gl_local();
    const double T = bc(y[0], 0);
    constexpr int st = 2 * NPT, NC = DERIV ? 19 : 15;
    // a row's coefficients: all read before the first is used (see Entry)
    auto row = [&](int a) { return tab + T_TH + (T < (mech::ONE_TMID ? mech::TMID : mech::PTMID[a]) ? 0 : NPT) + a; };
    double c[NC], iW[R];
    auto read = [&](int r) {
        const double* t = row(r * 16 + i);
#pragma unroll
        for (int k = 0; k < NC; ++k) c[k] = t[k * st];
    };
#pragma unroll
    for (int r = 0; r < R; ++r) iW[r] = mech::PW[NPT + r * 16 + i];        // 0 at T's position and past the last
    read(0);
    __builtin_amdgcn_sched_barrier(0);
    x.T = T;
    x.p = p;
    x.lnT = chem_math::ln(T);
    x.iT = chem_math::recip(T);
    const double T2 = T * T, T3 = T2 * T, T4 = T2 * T2;
    double sig = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        th.yw[r] = y[r] * iW[r];
        sig = sig + th.yw[r];
    }
#pragma unroll
    for (int q = 0; q < RI; ++q) sig = sig + ywi[q];
    sig = gsum(sig);
    th.sig = sig;
    th.Wbar = chem_math::recip(sig);
    th.rho = p * th.Wbar * x.iT * (1.0 / mech::RU);
    th.irho = mech::RU * T * sig * ip;
    x.ctot = p * x.iT * (1.0 / mech::RU);
    x.lnPRT = mech::LN_PATM_R - x.lnT;
    x.rtp = T * mech::RU_PATM;
    x.prt = x.iT * mech::PATM_RU;
    double cpm = 0.0, dcpm = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int a = r * 16 + i;
        if (r > 0) {
            read(r);
            __builtin_amdgcn_sched_barrier(0);
        }
        double v = T4 * c[4];
        v = fma(T3, c[3], v);
        v = fma(T2, c[2], v);
        v = fma(T, c[1], v);
        th.cpR[r] = v + c[0];
        v = T4 * c[8];
        v = fma(T3, c[7], v);
        v = fma(T2, c[6], v);
        v = fma(T, c[5], v);
        v = fma(x.iT, c[9], v);
        th.HRT[r] = v + c[0];
        v = T4 * c[13];
        v = fma(T3, c[12], v);
        v = fma(T2, c[11], v);
        v = fma(T, c[10], v);
        v = fma(x.lnT, c[0], v);
        v = fma(-x.iT, c[9], v);
        const double Gk = v + c[14];
        if constexpr (DERIV) {
            v = T3 * c[18];
            v = fma(T2, c[17], v);
            v = fma(T, c[16], v);
            th.dcpR[r] = v + c[15];
            dcpm = fma(th.dcpR[r], th.yw[r], dcpm);
        }
        cpm = fma(th.cpR[r], th.yw[r], cpm);
        if (a >= 1 && a < NACT) {
            const double gp = chem_math::exp_poly(Gk);
            L[L_C + a - 1] = th.rho * th.yw[r];
            L[L_GP + a - 1] = gp;
            L[L_GM + a - 1] = chem_math::recip(gp);
            L[L_H + a - 1] = th.HRT[r];
            if (mech::HAS_LNKC) L[L_G + a - 1] = Gk;
        }
    }
    // the species no reaction changes, and the neutral entry after the last:
    // they cancel between the sides of any reaction, so only C and cp matter
#pragma unroll
    for (int q = 0; q < RI; ++q) {
        const int m = q * 16 + i;
        const int a = R * 16 + m;
        const double* c = row(a);
        double v = T4 * c[4 * st];
        v = fma(T3, c[3 * st], v);
        v = fma(T2, c[2 * st], v);
        v = fma(T, c[1 * st], v);
        th.cpi[q] = v + c[0];
        cpm = fma(th.cpi[q], ywi[q], cpm);
        if (DERIV) {
            v = T3 * c[18 * st];
            v = fma(T2, c[17 * st], v);
            v = fma(T, c[16 * st], v);
            dcpm = fma(v + c[15 * st], ywi[q], dcpm);
        }
        if (m <= NI) {
            L[L_C + NA + m] = m < NI ? th.rho * ywi[q] : 1.0;
            L[L_GP + NA + m] = 1.0;
            L[L_GM + NA + m] = 1.0;
            L[L_H + NA + m] = 0.0;
            if (mech::HAS_LNKC) L[L_G + NA + m] = 0.0;
        }
    }
    th.cpm = gsum(cpm);
    if (DERIV) th.dcpm = gsum(dcpm);
}

// A list word: byte offset from the first reaction array | coefficient << 24.
__device__ __forceinline__ double list_value(const double* __restrict__ Q, int w)
{
    return *(const double*)((const char*)Q + (w & 0xffffff));
}
__device__ __forceinline__ double list_coef(int w) { return (double)(w >> 24); }

// A stream of list words.  Lists stay rolled loops (unrolled, the 32-species
// step was 220 KB of code, several times the instruction cache), LC lists side
// by side: row t of the table holds word t of each of them for the 16 lanes, a
// lane's words together (16-byte loads).
// run(len, use) walks the next len rows (an even number), calling use(q, w) for
// word w of list q.  The words are loaded two rows ahead, across the lists that
// follow one another in the table (which ends with two spare rows), so a stream
// begun before other work has its first words when it is walked.  The address
// passes through an empty asm, or the compiler would load whole tables ahead of
// the substep loop and spill them.
template <int LC>
struct Stream {
    typedef const __attribute__((address_space(1))) char gchar;
    typedef int int4v __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) int4v gint4;
    unsigned long long base;
    int4v w[2][LC / 4];

    __device__ __forceinline__ void words(int h)
    {
#pragma unroll
        for (int v = 0; v < LC / 4; ++v)
            w[h][v] = *(gint4*)((gchar*)base + 4u * LC * (unsigned)gl() + h * LC * 64 + v * 16);
    }
    __device__ __forceinline__ explicit Stream(const int* table)
    {
        base = (unsigned long long)table;
        asm volatile("" : "+s"(base));
        words(0);
        words(1);
    }
    // load(w) returns what use(q, coefficient, value) takes for the word w of
    // list q.  The loads of B rows are issued before their first use: left to
    // the compiler, every one is waited for by itself (two LDS round trips a
    // word with derivatives): the Jacobian lists of 16 species took 13,900
    // cycles, now 8,500.
    template <int B, class Load, class Use>
    __device__ __forceinline__ void run(int len, Load&& load, Use&& use)
    {
#pragma unroll 1
        for (int t = 0; t < len; t += 2) {
            base += 2 * LC * 64;
#pragma unroll
            for (int h = 0; h < 2; h += B) {
                decltype(load(0)) v[B][LC];
                int c[B][LC];
#pragma unroll
                for (int b = 0; b < B; ++b)
#pragma unroll
                    for (int q = 0; q < LC; ++q) {
                        const int k = w[h + b][q / 4][q % 4];
                        v[b][q] = load(k);
                        c[b][q] = k;
                    }
#pragma unroll
                for (int b = 0; b < B; ++b) words(h + b);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int b = 0; b < B; ++b)
#pragma unroll
                    for (int q = 0; q < LC; ++q) use(q, list_coef(c[b][q]), v[b][q]);
            }
        }
    }
};

// Source terms f (the lane's components) at the state y; with JAC the lane's
// rows of the Jacobian's first NC position columns in A.  Every lane of the
// group calls it together.
template <bool JAC, int NC>
__device__ __forceinline__ void rhs(const double* __restrict__ tab, double p, double ip, const double (&y)[R],
                                    const double (&ywi)[RI], double* __restrict__ L, double (&f)[R],
                                    double (&A)[R][NC])
{
    const int i = gl_local();
    Mix x;
    Thermo<JAC> th;
    if (i < NARR) L[L_A + i * NRW + NR] = 0.0;
    Stream<4> list(&mech::RL[0]);
    thermo<JAC>(tab, p, ip, y, ywi, L, x, th);
    lds_sync();
    double* const Q = L + L_A;
    auto store = [&](int j, const Rate& o) {
        Q[j] = o.q;
        if (JAC) {
            Q[NRW + j] = o.dqT;
            Q[2 * NRW + j] = o.s;
            Q[3 * NRW + j] = o.kf;
            Q[4 * NRW + j] = o.kr;
        }
    };
    // Rounds of 16 reactions; those after the first FULL_ROUNDS hold elementary
    // ones only and go two at a time, so one's arithmetic covers the other's.
    Entry next(tab, i);
#pragma unroll 1
    for (int j = i; j < 16 * mech::FULL_ROUNDS; j += 16) {
        const Entry en = next;
        const Slots<JAC> sl(en, L);
        next = Entry(tab, j + 16);
        __builtin_amdgcn_sched_barrier(0);
        if (j < NR) {
            Rate o;
            reaction<true, JAC>(en, sl, tab, L, x, o);
            store(j, o);
            const int misc = en.w[NWORDS - 1], kind = misc & 7;
            if (JAC && NTB > 0 && kind >= 1 && kind <= 4) {
                const int t = (misc >> 16) & 0xffff;
                L[L_X + t] = o.dM;
                for (int q = 0; q < MAXP; ++q) L[L_X + NTB + t * MAXP + q] = tab[T_TBC + q * NTB + t] * o.dM;
            }
        }
    }
    constexpr int ELEMENTARY = ROUNDS - mech::FULL_ROUNDS;
#pragma unroll 1
    for (int j = 16 * mech::FULL_ROUNDS + i; j < 16 * (mech::FULL_ROUNDS + ELEMENTARY / 2 * 2) ; j += 32) {
        const Entry e0 = next, e1(tab, j + 16);
        const Slots<JAC> s0(e0, L);
        const Slots<JAC> s1(e1, L);
        next = Entry(tab, j + 32);
        __builtin_amdgcn_sched_barrier(0);
        Rate o0, o1;
        reaction<false, JAC>(e0, s0, tab, L, x, o0);
        reaction<false, JAC>(e1, s1, tab, L, x, o1);
        if (j < NR) store(j, o0);
        if (j + 16 < NR) store(j + 16, o1);
    }
    if constexpr (ELEMENTARY % 2 != 0) {
        const int j = 16 * (ROUNDS - 1) + i;
        const Slots<JAC> sl(next, L);
        __builtin_amdgcn_sched_barrier(0);
        Rate o;
        reaction<false, JAC>(next, sl, tab, L, x, o);
        if (j < NR) store(j, o);
    }
    lds_sync();
    double wd[R], wT[R], Sk[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wd[r] = wT[r] = Sk[r] = 0.0;
    static_for<0, R>([&](auto rc) {
        constexpr int r = decltype(rc)::v;
        struct Values {
            double q, T, s;
        };
        auto load = [&](int w) {
            Values v;
            v.q = list_value(Q, w);
            if (JAC) {
                v.T = list_value(Q + NRW, w);
                v.s = list_value(Q + 2 * NRW, w);
            }
            return v;
        };
        list.template run<JAC ? 1 : 2>(mech::WLEN[r], load, [&](int, double nu, const Values& v) {
            wd[r] = fma(nu, v.q, wd[r]);
            if (JAC) {
                wT[r] = fma(nu, v.T, wT[r]);
                Sk[r] = fma(nu, v.s, Sk[r]);
            }
        });
    });
    double hw = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) hw = fma(th.HRT[r], wd[r], hw);     // T's position has no terms: wd = 0
    hw = gsum(hw);
    const double icpm = chem_math::recip(th.cpm);
    const double rcpinv = x.T * th.sig * ip * icpm;
    const double fT = -mech::RU * x.T * hw * rcpinv;
#pragma unroll
    for (int r = 0; r < R; ++r) f[r] = mech::PW[r * 16 + i] * (th.irho * wd[r]);
    f[0] = i == 0 ? fT : f[0];
    if constexpr (JAC) {
        lds_sync();
        // the partials d q / d C of every slot, over the arrays just read (a
        // reaction's rate constants are read before its own words of the
        // arrays they sit in are overwritten)
        const int* const words = (const int*)(tab + T_INT) + I_WORDS;
        Stream<mech::JGW> cols(&mech::JL[0]);
#pragma unroll 2
        for (int j = i; j < NR; j += 16) {
            int ra[MOLR], pa[MOLP];
#pragma unroll
            for (int s = 0; s < MOLR; ++s) ra[s] = (words[(s / 4) * NR + j] >> (8 * (s % 4))) & 255;
#pragma unroll
            for (int s = 0; s < MOLP; ++s) pa[s] = (words[(WR + s / 4) * NR + j] >> (8 * (s % 4))) & 255;
            const double kf = Q[3 * NRW + j], kr = Q[4 * NRW + j];
#pragma unroll
            for (int s = 0; s < MOLR; ++s) Q[s * NRW + j] = others<MOLR>(L, ra, s, kf);
#pragma unroll
            for (int s = 0; s < MOLP; ++s) Q[(MOLR + s) * NRW + j] = others<MOLP>(L, pa, s, -kr);
        }
        lds_sync();
        // concentration Jacobian Jc_km = d wdot_k / d C_m: the third-body part
        // common to all columns, then each column's slots and corrections
        double D[R], own[R];
        auto value = [&](int w) { return list_value(Q, w); };
        static_for<0, R>([&](auto rc) {
            constexpr int r = decltype(rc)::v;
            D[r] = 0.0;
            list.template run<2>(mech::DLEN[r], value, [&](int, double c, double v) { D[r] = fma(c, v, D[r]); });
        });
        static_for<0, R>([&](auto rc) {
            constexpr int r = decltype(rc)::v;
            own[r] = D[r];
            list.template run<2>(mech::DGLEN[r], value, [&](int, double c, double v) { own[r] = fma(c, v, own[r]); });
        });
        // (columns in groups of similar list length, those of the step's
        // unknowns first)
        static_for<0, NC == NACT ? mech::JGACT : mech::JGALL>([&](auto gc) {
            constexpr int g = decltype(gc)::v, r = mech::JGROW[g];
            double acc[mech::JGW];
#pragma unroll
            for (int q = 0; q < mech::JGW; ++q) acc[q] = D[r];
            cols.template run<1>(mech::JGLEN[g], value, [&](int q, double c, double v) { acc[q] = fma(c, v, acc[q]); });
            static_for<0, mech::JGW>([&](auto qc) {
                constexpr int q = decltype(qc)::v, m = mech::JGCOL[g * mech::JGW + q];
                if constexpr (m >= 0) A[r][1 + m] = m < NA && (m + 1) / 16 == r && (m + 1) % 16 == i ? own[r] : acc[q];
            });
        });
        // chain rule to (T, Y), with S_k = sum_l Jc_kl C_l:
        //   J_km = (W_k/W_m) Jc_km + (Wbar/W_m)(f_k - W_k S_k / rho)
        //   J_k0 = (W_k / rho)(wT_k - S_k / T) + f_k / T
        //   J_0m = -R T (rho HJ_m - Wbar HS) / (W_m rho cp) - f_T (cp_m / cp - Wbar / W_m)
        //   J_00 = -R (cpw + T HwT - HS) / (rho cp) - f_T (dcp / cp - 1/T)
        // HJ_m = sum_k H_k/RT Jc_km, HS = sum_k H_k/RT S_k, HwT = sum_k H_k/RT wT_k,
        // cpw = sum_k cp_k/R wdot_k
        double HS = 0.0, HwT = 0.0, cpw = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            HS = fma(th.HRT[r], Sk[r], HS);
            HwT = fma(th.HRT[r], wT[r], HwT);
            cpw = fma(th.cpR[r], wd[r], cpw);
        }
        HS = gsum(HS);
        HwT = gsum(HwT);
        cpw = gsum(cpw);
        const double RT = mech::RU * x.T;
        const double icp = icpm * (1.0 / mech::RU);
        const double dcp = mech::RU * th.dcpm;
        double wg[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double W = mech::PW[r * 16 + i];
            wg[r] = th.Wbar * fma(-W, Sk[r] * th.irho, f[r]);
            A[r][0] = fma(W * th.irho, wT[r] - Sk[r] * x.iT, f[r] * x.iT);
        }
        const double J00 = -mech::RU * (cpw + x.T * HwT - HS) * rcpinv - fT * (dcp * icp - x.iT);
        A[0][0] = i == 0 ? J00 : A[0][0];
        // (static_for: a pragma stops unrolling above some 45 columns, and the rows
        // then sit in scratch memory)
        static_for<0, NC - 1>([&](auto mc) {
            constexpr int m = decltype(mc)::v;
            double HJ = 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r) HJ = fma(th.HRT[r], A[r][1 + m], HJ);
            HJ = gsum(HJ);
            // cp/R of species m, from the lane that holds its position
            const double cpm_m = m < NA ? bc(th.cpR[(m + 1) / 16 < R ? (m + 1) / 16 : 0], (m + 1) % 16)
                                        : bc(th.cpi[m >= NA ? (m - NA) / 16 : 0], (m - NA) % 16);
            const double iW = mech::IWM[m];
            const double t = fma(th.rho, HJ, -th.Wbar * HS) * (-RT * rcpinv);
            const double u = fma(cpm_m, icp * mech::RU, -th.Wbar);
            const double J0m = fma(-fT, u, t) * iW;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int a = r * 16 + i;
                double v = fma(A[r][1 + m], mech::PW[a], wg[r]) * iW;
                if (r == 0) v = i == 0 ? J0m : v;
                if (r * 16 + 15 >= NACT) v = a < NACT ? v : 0.0;
                A[r][1 + m] = v;
            }
        });
        if (R * 16 > NACT) A[R - 1][0] = (R - 1) * 16 + i < NACT ? A[R - 1][0] : 0.0;
    }
}

// ---- linear algebra of the group's NACT x NACT matrix ----
// A: rows by position; after lu() the multipliers below the diagonal (zero in
// the lanes on and above it within the diagonal blocks), and above it the
// rows of U divided by their pivots; U's diagonal blocks in UD; D: 1 / pivot.
// Row interchanges move whole rows, so a solve permutes its right-hand side
// once (src: the position whose row came here).
struct Factors {
    double A[R][NACT];
    double UD[R][16];
    double D[R];
    int src[R];
    bool swapped;
};

// LU with partial pivoting (the lowest position among equal magnitudes).
__device__ __forceinline__ void lu(Factors& F, bool& ok)
{
    const int i = gl_local();
    ok = true;
    F.swapped = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        F.src[r] = r * 16 + i;
        F.D[r] = 0.0;
    }
    static_for<0, NACT>([&](auto kc) {
        constexpr int k = decltype(kc)::v, rk = k / 16, lk = k % 16;
        double v[R], vm = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = -1.0;
#pragma unroll
        for (int r = rk; r < R; ++r) {
            v[r] = fabs(F.A[r][k]);
            if (r == rk) v[r] = i >= lk ? v[r] : -1.0;
            vm = r == rk ? v[r] : fmax(vm, v[r]);
        }
        const double vmax = gmax(vm);
        ok = ok && (vmax > 0.0);
        // rows move only if some cell's largest entry is not on the diagonal
        const unsigned long long diag = 0x0001000100010001ull << lk;
        const unsigned long long here = __ballot(v[rk] == vmax) & diag;
        if (here != (__ballot(true) & diag)) {
            F.swapped = true;
            int idx = k;
            bool found = false;
#pragma unroll
            for (int r = rk; r < R; ++r) {
                const unsigned bits = (unsigned)(__ballot(v[r] == vmax) >> gbase()) & 0xffffu;
                if (!found && bits) {
                    idx = r * 16 + __builtin_ctz(bits);
                    found = true;
                }
            }
            if (!(vmax > 0.0)) idx = k;
            const int li = idx & 15, ri = idx >> 4;
#pragma unroll
            for (int c = 0; c < NACT; ++c) {
                double s = F.A[rk][c];
#pragma unroll
                for (int r = rk + 1; r < R; ++r) s = ri == r ? F.A[r][c] : s;
                const double top = bc(F.A[rk][c], lk), low = gather(s, li);
#pragma unroll
                for (int r = rk; r < R; ++r) F.A[r][c] = (i == li && ri == r) ? top : F.A[r][c];
                F.A[rk][c] = i == lk ? low : F.A[rk][c];
            }
            {
                int s = F.src[rk];
#pragma unroll
                for (int r = rk + 1; r < R; ++r) s = ri == r ? F.src[r] : s;
                const int top = __shfl(F.src[rk], gbase() + lk, 64), low = __shfl(s, gbase() + li, 64);
#pragma unroll
                for (int r = rk; r < R; ++r) F.src[r] = (i == li && ri == r) ? top : F.src[r];
                F.src[rk] = i == lk ? low : F.src[rk];
            }
        }
        const double rp = chem_math::recip(bc(F.A[rk][k], lk));
        double l[R];
#pragma unroll
        for (int r = rk; r < R; ++r) {
            l[r] = F.A[r][k] * rp;
            if (r == rk) l[r] = i > lk ? l[r] : 0.0;
        }
        F.D[rk] = i == lk ? rp : F.D[rk];
#pragma unroll
        for (int c = k + 1; c < NACT; ++c) {
            const double pc = bc(F.A[rk][c], lk);
#pragma unroll
            for (int r = rk; r < R; ++r) F.A[r][c] = fma(-l[r], pc, F.A[r][c]);
        }
        // column k: the multipliers below, U above (rows of this block only)
#pragma unroll
        for (int r = rk; r < R; ++r) F.A[r][k] = r == rk ? (i > lk ? l[r] : F.A[r][k]) : l[r];
    });
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int c = 0; c < NACT; ++c) {
            const int rc = c / 16, lc = c % 16;
            if (rc == r) {
                F.UD[r][lc] = i < lc ? F.A[r][c] * F.D[r] : 0.0;
                F.A[r][c] = i > lc ? F.A[r][c] : 0.0;
            } else if (rc > r) {
                F.A[r][c] = F.A[r][c] * F.D[r];
            }
        }
    }
}

// b[r] <- b at position src[r]
__device__ __forceinline__ void permute(const int (&src)[R], double (&b)[R])
{
    double n[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        n[r] = gather(b[0], src[r] & 15);
#pragma unroll
        for (int q = 1; q < R; ++q) {
            const double g = gather(b[q], src[r] & 15);
            n[r] = (src[r] >> 4) == q ? g : n[r];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) b[r] = n[r];
}

// Solve M x = b for the group's vector b.
__device__ __forceinline__ void solve(const Factors& F, double (&b)[R])
{
    if (F.swapped) permute(F.src, b);
    static_for<0, NACT - 1>([&](auto kc) {
        constexpr int k = decltype(kc)::v, rk = k / 16;
        const double z = bc(b[rk], k % 16);
#pragma unroll
        for (int r = rk; r < R; ++r) b[r] = fma(-F.A[r][k], z, b[r]);
    });
#pragma unroll
    for (int r = 0; r < R; ++r) b[r] *= F.D[r];
    static_for<0, NACT - 1>([&](auto kc) {
        constexpr int k = NACT - 1 - decltype(kc)::v, rk = k / 16;
        const double z = bc(b[rk], k % 16);
#pragma unroll
        for (int r = 0; r <= rk; ++r) b[r] = fma(r == rk ? -F.UD[r][k % 16] : -F.A[r][k], z, b[r]);
    });
}

// One RODAS4 step from y with step h; false if the step matrix is singular or
// a result is not finite.  L: the cell's scratch.
__device__ __forceinline__ bool ros_step(const double* __restrict__ tab, double p, double ip, const double (&y)[R],
                                         const double (&ywi)[RI], const double (&yi)[RI], double h, double rtol,
                                         double atol, double* __restrict__ L, double (&ynew)[R], double& errn)
{
    const int i = gl_local();
    Factors F;
    double u[Rodas4::S - 1][R], f[R], us[R];
    rhs<true, NACT>(tab, p, ip, y, ywi, L, f, F.A);
    const double hinv = chem_math::recip(h);
    const double ghinv = hinv * (1.0 / Rodas4::gamma);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < NACT; ++c) F.A[r][c] = (r * 16 + i == c ? ghinv : 0.0) - F.A[r][c];
    bool ok;
    lu(F, ok);
    solve(F, f);
#pragma unroll
    for (int s = 0; s < Rodas4::S - 1; ++s)
#pragma unroll
        for (int r = 0; r < R; ++r) u[s][r] = s == 0 ? f[r] : 0.0;
    // one copy of the source-term code for the five later stages (the kernel
    // stays inside the instruction cache); stage vectors stay in registers
#pragma unroll 1
    for (int s = 1; s < Rodas4::S; ++s) {
        double Ys[R], acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            Ys[r] = y[r];
            acc[r] = 0.0;
        }
        // (the tableau's rows are zero from the stage on, as are the vectors)
#pragma unroll
        for (int j = 0; j < Rodas4::S - 1; ++j) {
            const double ra = RA[s][j], rc = RC[s][j];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                Ys[r] = fma(ra, u[j][r], Ys[r]);
                acc[r] = fma(rc, u[j][r], acc[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) ynew[r] = Ys[r];        // the last stage's: y_new = Y_6 + u_6
        double none[R][1];
        rhs<false, 1>(tab, p, ip, Ys, ywi, L, us, none);
#pragma unroll
        for (int r = 0; r < R; ++r) us[r] = fma(acc[r], hinv, us[r]);
        solve(F, us);
#pragma unroll
        for (int j = 1; j < Rodas4::S - 1; ++j)
            if (j == s)
#pragma unroll
                for (int r = 0; r < R; ++r) u[j][r] = us[r];
    }
    double e2 = 0.0;
    bool bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        ynew[r] += us[r];
        const double sc = atol + rtol * fmax(fabs(y[r]), fabs(ynew[r]));
        const double e = us[r] * chem_math::recip(sc);
        const bool in = r * 16 + i < NACT;
        e2 = in ? fma(e, e, e2) : e2;
        bad = bad || (in && !finite(ynew[r]));
    }
    // species no reaction changes have no error, except that a zero scale
    // fails the step (0 / 0) as it does in any other component
#pragma unroll
    for (int q = 0; q < RI; ++q) {
        const double e = 0.0 * chem_math::recip(atol + rtol * fabs(yi[q]));
        if (q * 16 + i < NI) e2 = fma(e, e, e2);
    }
    errn = sqrt(gsum(e2) * (1.0 / N));
    return ok && !gany(bad) && finite(errn);
}

// Per-group integration state (the lane's components, the rest replicated).
struct Cell {
    double y[R], yi[RI], ywi[RI];
    double p, ip, t, h;
    int nacc, nrej, status;
    bool rej_last, done;
};

__device__ __forceinline__ void cell_begin(Cell& c, double T, double p, const double* __restrict__ Y, double h0)
{
    const int i = gl();
    bool bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int k = mech::PSPEC[r * 16 + i];
        c.y[r] = k >= 0 ? Y[k] : 0.0;
        if (r == 0 && i == 0) c.y[r] = T;
        bad = bad || !finite(c.y[r]);
    }
#pragma unroll
    for (int q = 0; q < RI; ++q) {
        const int k = mech::PSPEC[R * 16 + q * 16 + i];
        c.yi[q] = k >= 0 ? Y[k] : 0.0;
        c.ywi[q] = c.yi[q] * mech::PW[NPT + R * 16 + q * 16 + i];
        bad = bad || !finite(c.yi[q]);
    }
    c.p = p;
    c.ip = 1.0 / p;
    c.t = 0.0;
    c.h = h0;
    c.nacc = 0;
    c.nrej = 0;
    c.rej_last = false;
    bad = gany(bad) || !(T > 0.0) || !(p > 0.0) || !finite(p);
    c.status = bad ? chem::CELL_BADINPUT : chem::CELL_OK;
    c.done = bad;
}

// One attempted substep with the controller of the one-cell-per-lane form;
// returns the step size if the step was accepted, else 0.
__device__ __forceinline__ double cell_attempt(Cell& c, const double* __restrict__ tab, const StepArgs& a,
                                               double* __restrict__ L)
{
    if (c.done) return 0.0;
    if (c.nacc + c.nrej >= a.max_substeps) {
        c.status = chem::CELL_MAXSTEPS;
        c.done = true;
        return 0.0;
    }
    if (c.h < a.hmin) {
        c.status = chem::CELL_HMIN;
        c.done = true;
        return 0.0;
    }
    bool last = false;
    double h = c.h;
    if (h >= a.dt - c.t) {
        h = a.dt - c.t;
        last = true;
    }
    double ynew[R], en;
    const bool ok = ros_step(tab, c.p, c.ip, c.y, c.ywi, c.yi, h, a.rtol, a.atol, L, ynew, en);
    if (ok && en <= 1.0) {
#pragma unroll
        for (int r = 0; r < R; ++r) c.y[r] = ynew[r];
        c.t = last ? a.dt : c.t + h;
        double fac = 0.9 * chem::inv_root4(fmax(en, 1e-16));
        fac = fmin(6.0, fmax(0.2, fac));
        if (c.rej_last) fac = fmin(1.0, fac);
        c.h = h * fac;
        c.rej_last = false;
        ++c.nacc;
        if (last) c.done = true;
        return h;
    }
    ++c.nrej;
    c.h = h * (ok ? fmax(0.2, 0.9 * chem::inv_root4(en)) : 0.2);
    c.rej_last = true;
    return 0.0;
}

// the lane's components of a state-sized vector to out[0] (T) and out_Y
__device__ __forceinline__ void put(const double (&y)[R], const double (&yi)[RI], double* __restrict__ T,
                                    double* __restrict__ Y)
{
    const int i = gl();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int k = mech::PSPEC[r * 16 + i];
        if (k >= 0) Y[k] = y[r];
        if (r == 0 && i == 0) *T = y[0];
    }
#pragma unroll
    for (int q = 0; q < RI; ++q) {
        const int k = mech::PSPEC[R * 16 + q * 16 + i];
        if (k >= 0) Y[k] = yi[q];
    }
}

__device__ __forceinline__ void cell_store(const Cell& c, double* __restrict__ T, double* __restrict__ Y, long cell,
                                           int* status, int* nacc, int* nrej)
{
    if (c.status != chem::CELL_BADINPUT) put(c.y, c.yi, T + cell, Y + cell * NS);
    if (gl() == 0) {   // the per-cell counters only where someone reads them (null: not asked for)
        if (status) status[cell] = c.status;
        if (nacc) nacc[cell] = c.nacc;
        if (nrej) nrej[cell] = c.nrej;
    }
}

// Groups of a workgroup: cpw of each wave hold a cell (the others have no
// scratch and leave).  The group's place among the launch's, or -1, and its
// scratch.
__device__ __forceinline__ long group_of(int cpw, int words, double* __restrict__ lds, double*& L)
{
    const int wave = (int)threadIdx.x / 64, grp = ((int)threadIdx.x & 63) / G;
    const int own = wave * cpw + grp;
    L = lds + TAB_DOUBLES + own * words;
    return grp < cpw ? (long)blockIdx.x * ((int)blockDim.x / 64 * cpw) + own : -1;
}

}  // namespace chemw

// ---- plain form: one group of 16 lanes per cell, cells in index order ----
// A field larger than the chip holds at once is dealt through one counter
// (a.head): a group takes the next cell when its own is done.  Dealt by the
// grid instead, a workgroup's groups wait for its slowest cell, and a front
// that runs along a grid line puts all the costly workgroups on the same few
// XCDs (workgroups go to the XCDs in turn).
extern "C" __global__ void __launch_bounds__(256, mech::WPS) chem_plain(chem::IntegrateArgs a)
{
    using namespace chemw;
    extern __shared__ double lds[];
    load_tables(lds, a.par);
    double* L;
    long cell = group_of(mech::CPW, mech::LDS_CELL, lds, L);
    if (cell < 0) return;
    Cell c;
    c.done = true;
    bool have = false, more = true;
    while (true) {
        if (!have && more) {
            if (a.head) {
                unsigned long long t = 0ull;
                if (gl() == 0) t = atomicAdd(a.head, 1ull);
                cell = (long)__shfl((long long)t, gbase(), 64);
            }
            have = cell < a.ncell;
            more = a.head && have;
            if (have) cell_begin(c, a.T[cell], a.p[cell], a.Y + cell * NS, a.h0 ? a.h0[cell] : a.step.dt);
        }
        if (__all(!have && !more)) break;
        if (have) {
            cell_attempt(c, lds, a.step, L);
            if (c.done) {
                cell_store(c, a.T, a.Y, cell, a.status, a.nacc, a.nrej);
                have = false;
            }
        }
    }
}

// ---- source terms and Jacobian at given states ----
extern "C" __global__ void __launch_bounds__(256, mech::WPS) chem_eval(EvalArgs a)
{
    using namespace chemw;
    extern __shared__ double lds[];
    load_tables(lds, a.par);
    double* L;
    const long first = group_of(mech::CPW, mech::LDS_CELL, lds, L);
    if (first < 0) return;
    const int i = gl();
    // the launch holds at most the resident workgroups, which share out the cells
    for (long cell = first; cell < a.ncell; cell += (long)gridDim.x * ((int)blockDim.x / 64 * mech::CPW)) {
        Cell c;
        cell_begin(c, a.T[cell], a.p[cell], a.Y + cell * NS, 0.0);
        double f[R];
        // what the species no reaction changes get: zero, or NaN in a state (a
        // Jacobian) that is not finite, as in every other component
        double zero[RI], z = fma(0.0, c.ip, 0.0);
#pragma unroll
        for (int r = 0; r < R; ++r) z = fma(0.0, c.y[r], z);
#pragma unroll
        for (int q = 0; q < RI; ++q) z = fma(0.0, c.yi[q], z);
        z = gsum(z);
#pragma unroll
        for (int q = 0; q < RI; ++q) zero[q] = z;
        if (a.J) {
            double A[R][N];
            rhs<true, N>(lds, c.p, c.ip, c.y, c.ywi, L, f, A);
            double za = 0.0;
            static_for<0, N>([&](auto cc) {
                constexpr int col = decltype(cc)::v;
#pragma unroll
                for (int r = 0; r < R; ++r) za = fma(0.0, A[r][col], za);
            });
            za = gsum(za);
            double* const J = a.J + cell * N * N;
#pragma unroll
            for (int r = 0; r < R + RI; ++r) {
                const int k = mech::PSPEC[r * 16 + i];
                const int row = r == 0 && i == 0 ? 0 : 1 + k;
                if (row > 0 || (r == 0 && i == 0)) {
                    static_for<0, N>([&](auto cc) {
                        constexpr int col = decltype(cc)::v;
                        const int oc = col == 0 ? 0 : 1 + mech::COLSPEC[col - 1];
                        J[row * N + oc] = r < R ? A[r < R ? r : 0][col] : za;
                    });
                }
            }
        } else {
            double none[R][1];
            rhs<false, 1>(lds, c.p, c.ip, c.y, c.ywi, L, f, none);
        }
        put(f, zero, a.f + cell * N, a.f + cell * N + 1);
    }
}

// ---- one fixed RODAS4 step of size h per cell (y_new and the error norm) ----
struct FixedStepArgs {
    const double* par;
    const double* T;
    const double* p;
    const double* Y;
    long ncell;
    double h;
    double* ynew;   // [ncell][N]
    double* err;    // [ncell]
    double rtol, atol;
    int* ok;
};

extern "C" __global__ void __launch_bounds__(256, mech::WPS) chem_fixed_step(FixedStepArgs a)
{
    using namespace chemw;
    extern __shared__ double lds[];
    load_tables(lds, a.par);
    double* L;
    const long cell = group_of(mech::CPW, mech::LDS_CELL, lds, L);
    if (cell < 0 || cell >= a.ncell) return;
    Cell c;
    cell_begin(c, a.T[cell], a.p[cell], a.Y + cell * NS, a.h);
    double yn[R], en;
    const bool ok = ros_step(lds, c.p, c.ip, c.y, c.ywi, c.yi, a.h, a.rtol, a.atol, L, yn, en);
    // where the step fails, the species no reaction changes fail with the others
    bool bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) bad = bad || (r * 16 + gl() < NACT && !finite(yn[r]));
    if (gany(bad))
#pragma unroll
        for (int q = 0; q < RI; ++q) c.yi[q] = __builtin_nan("");
    put(yn, c.yi, a.ynew + cell * N, a.ynew + cell * N + 1);
    if (gl() == 0) {
        a.err[cell] = en;
        a.ok[cell] = ok ? 1 : 0;
    }
}

// ---- persistent form: groups pull cells from one global counter ----
// Cells of all fields form one index space [0, total); each group takes the
// next cell when its current one is done, so no group idles while cells
// remain (the hardware already balances whole waves; this also balances the
// groups inside a wave and spans several fields in one launch).
extern "C" __global__ void __launch_bounds__(256, mech::WPS) chem_persistent(const PersistBlock* __restrict__ blk,
                                                                         unsigned long long* __restrict__ heads,
                                                                         const double* __restrict__ par)
{
    using namespace chemw;
    extern __shared__ double lds[];
    load_tables(lds, par);
    double* L;
    if (group_of(mech::CPW, mech::LDS_CELL, lds, L) < 0) return;
    const StepArgs step = blk->step;
    const long total = blk->total;
    Cell c;
    c.done = true;
    bool have = false, exhausted = false;
    long local = 0;
    int f = 0;
    while (true) {
        if (!have && !exhausted) {
            unsigned long long t = 0ull;
            if (gl() == 0) t = atomicAdd(heads, 1ull);
            t = (unsigned long long)__shfl((long long)t, gbase(), 64);
            if ((long)t < total) {
                f = field_of(blk, (long)t);
                const FieldDesc& fd = blk->fields[f];
                local = (long)t - fd.start;
                cell_begin(c, fd.T[local], fd.p[local], fd.Y + local * NS, step.dt);
                have = true;
            } else {
                exhausted = true;
            }
        }
        if (__all(exhausted && !have)) break;
        if (have) {
            cell_attempt(c, lds, step, L);
            if (c.done) {
                const FieldDesc& fd = blk->fields[f];
                cell_store(c, fd.T, fd.Y, local, fd.status, fd.nacc, fd.nrej);
                have = false;
            }
        }
    }
}
