// wide_rows.hip -- the forward kernels of the row-per-lane form, after
// wide_adjoint.hip, whose step and cell functions they run.
//
// The form of the mechanisms the 16-lane form of wide.hip is not the better one
// for: above 48 unknowns, where a lane would own four matrix rows and the step
// spills 1.9 KB a lane (48 reacting species, 238 reactions: a 65,536-cell field
// 28 ms there, 20-23 ms here; one cell 0.30 against 0.18-0.20), and those whose
// tables and scratch do not fit the LDS in that form (1,782 reactions).  Up to
// 48 unknowns the 16-lane form is the faster one, spilling or not: 6.5-7.1 ms
// against 10.2-10.9 at 34 species, 13.7 against 20-23 at 48 with 46 reacting,
// 59 against 90-114 at 34 with 972 reactions.  (Jacobians alone are 8 % slower
// there at 45 species and 12-20 % from a thousand reactions on.)

// ---- plain form: one group of G lanes per cell, cells in index order ----
extern "C" __global__ void __launch_bounds__(64, 2) chem_plain(chem::IntegrateArgs a)
{
    using namespace chemw;
    extern __shared__ double lds[];
    const int grp = (int)threadIdx.x / G;
    const long cell = (long)blockIdx.x * CPW + grp;
    if (cell >= a.ncell) return;
    double* L = lds + grp * mech::LDS_CELL;
    Cell c;
    cell_begin(c, a.T[cell], a.p[cell], a.Y + cell * NS, a.h0 ? a.h0[cell] : a.step.dt);
    while (!c.done) cell_attempt(c, a.par, a.step, L, L + mech::L_J);
    cell_store(c, a.T, a.Y, cell, a.status, a.nacc, a.nrej);
}

// ---- source terms and Jacobian at given states ----
extern "C" __global__ void __launch_bounds__(64) chem_eval(EvalArgs a)
{
    using namespace chemw;
    extern __shared__ double lds[];
    const int grp = (int)threadIdx.x / G;
    const long cell = (long)blockIdx.x * CPW + grp;
    if (cell >= a.ncell) return;
    double* L = lds + grp * mech::LDS_CELL;
    const int i = gl();
    const double p = a.p[cell];
    const double yi = i == 0 ? a.T[cell] : (i <= NS ? a.Y[cell * NS + i - 1] : 0.0);
    double A[N];
    double g[ROUNDS][3];
    double f;
    if (a.J) {
        f = rhs<double, F_JAC>(a.par, p, 1.0 / p, yi, L, A, 0.0, g);
        if (i < N) {
#pragma unroll
            for (int j = 0; j < N; ++j) a.J[(cell * N + i) * N + j] = A[j];
        }
    } else {
        f = rhs<double, F_ONLY>(a.par, p, 1.0 / p, yi, L, A, 0.0, g);
    }
    if (i < N) a.f[cell * N + i] = f;
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

extern "C" __global__ void __launch_bounds__(64) chem_fixed_step(FixedStepArgs a)
{
    using namespace chemw;
    extern __shared__ double lds[];
    const int grp = (int)threadIdx.x / G;
    const long cell = (long)blockIdx.x * CPW + grp;
    if (cell >= a.ncell) return;
    double* L = lds + grp * mech::LDS_CELL;
    const int i = gl();
    const double p = a.p[cell];
    const double yi = i == 0 ? a.T[cell] : (i <= NS ? a.Y[cell * NS + i - 1] : 0.0);
    double yn, en;
    const bool ok = ros_step(a.par, p, 1.0 / p, yi, a.h, a.rtol, a.atol, L, L + mech::L_J, yn, en);
    if (i < N) a.ynew[cell * N + i] = yn;
    if (i == 0) {
        a.err[cell] = en;
        a.ok[cell] = ok ? 1 : 0;
    }
}

// ---- persistent form: groups pull cells from one global counter ----
// Cells of all fields form one index space [0, total); each group takes the
// next cell when its current one is done, so no group idles while cells
// remain (the hardware already balances whole waves; this also balances the
// groups inside a wave and spans several fields in one launch).
extern "C" __global__ void __launch_bounds__(64, 2) chem_persistent(const PersistBlock* __restrict__ blk,
                                                                 unsigned long long* __restrict__ heads,
                                                                 const double* __restrict__ par)
{
    using namespace chemw;
    extern __shared__ double lds[];
    const int grp = (int)threadIdx.x / G;
    double* L = lds + grp * mech::LDS_CELL;
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
        if (__all(exhausted)) break;
        if (have) {
            cell_attempt(c, par, step, L, L + mech::L_J);
            if (c.done) {
                const FieldDesc& fd = blk->fields[f];
                cell_store(c, fd.T, fd.Y, local, fd.status, fd.nacc, fd.nrej);
                have = false;
            }
        }
    }
}
