// codegen.hpp -- mechanism-specific device source generation.
#pragma once

#include <cstdint>
#include <string>

#include "mechanism.hpp"

namespace chemmi {

// HIP source of namespace mech { NS, NR, N, rhs(), rhs_jac(), jtv_param() } for
// m: straight-line code for the one-cell-per-lane kernels.
std::string generate_mechanism_source(const MechanismData& m);

// Unknowns of a step: T and the species some reaction changes.
int active_unknowns(const MechanismData& m);

// Layout of the wave-cooperative form: 16 lanes per cell, lane i owning the
// positions r * 16 + i (T, then the species some reaction changes), and the
// per-cell LDS scratch in doubles.
struct WideLayout {
    int G = 16;            // lanes per cell (0: the mechanism does not fit the form)
    int na = 0;            // species some reaction changes
    int r = 1, ri = 1;     // positions a lane owns; of the other species (and a neutral entry)
    int molr = 1, molp = 1;   // most species slots on a reaction's sides
    int ntb = 0, maxp = 0; // reactions with a third body, most partners of efficiency other than 1
    bool lnkc = false;     // some reaction's K_c leaves the range of the per-species factors
    int cpw = 4;           // cells per wave
    int wpb = 4;           // waves per workgroup
    int table = 0;         // doubles of a workgroup's tables
    int lds_cell = 0;      // doubles per cell
    // Waves per SIMD the kernels' registers are shared by: a lane's rows of the
    // matrix and of its factors fit half the registers at one row a lane, and
    // need them all from two on.
    int waves_per_simd() const { return r == 1 ? 2 : 1; }
    int block() const { return 64 * wpb; }
    unsigned lds_bytes() const { return (unsigned)((table + wpb * cpw * lds_cell) * sizeof(double)); }
    // resident workgroups per compute unit, by registers and by LDS (160 KB)
    int blocks_per_cu() const
    {
        const int by_lds = (int)(160u * 1024u / lds_bytes()), by_regs = 4 * waves_per_simd() / wpb;
        return by_lds < 1 ? 1 : by_lds < by_regs ? by_lds : by_regs;
    }
    // The form is the better one where it fits: a lane owns at most three
    // matrix rows (measured where the row-per-lane kernels are), and one cell's
    // scratch and the tables fit the LDS.
    bool better() const { return r <= 3 && lds_bytes() <= 160u * 1024u; }
};

// The layout for m, or an empty optional-like result (G = 0) if m does not
// fit the form (more than 3 terms or a coefficient above 3 on a reaction
// side, or a table field too narrow).
WideLayout wide_layout(const MechanismData& m);

// HIP source of namespace mech for the wave-cooperative kernels: sizes,
// layout constants and the thermo, reaction and species tables they read.
std::string generate_wide_source(const MechanismData& m, const WideLayout& w);

// Layout of the wave-cooperative adjoint: G lanes per cell (a power of two >= n),
// and the per-cell LDS scratch in doubles.
struct RowLayout {
    int G = 64;
    int maxt = 1;          // most terms on one side of a reaction
    int nslot = 2;         // species partial slots per reaction (2 maxt)
    int pw = 4;            // doubles per reaction in the partials block
    int jw = 1;            // row stride of the concentration Jacobian (odd)
    int l_y = 0, l_c = 0, l_g = 0, l_h = 0, l_q = 0, l_p = 0, l_j = 0, l_t0 = 0, l_w = 0;
    int lds_cell = 0;      // doubles per cell
    int adj_lds_cell = 0;  // doubles per cell in the adjoint: the scratch for dual numbers,
                           // then the pivot row and indices (untouched by source evaluations)
    int cells_per_wave() const { return 64 / G; }
    // resident waves per compute unit of the forward kernels, by registers and LDS
    int blocks_per_cu() const
    {
        const int by_lds = (int)(160u * 1024u / lds_bytes());
        return by_lds < 1 ? 1 : by_lds < 8 ? by_lds : 8;
    }
    unsigned lds_bytes() const { return (unsigned)(cells_per_wave() * lds_cell * sizeof(double)); }
    unsigned adj_lds_bytes() const { return (unsigned)(cells_per_wave() * adj_lds_cell * sizeof(double)); }
};

// The layout for m, or an empty optional-like result (G = 0) if m does not
// fit the form (n > 64, or more than 3 terms on a reaction side).
RowLayout row_layout(const MechanismData& m);

// HIP source of namespace mech for the wave-cooperative adjoint: sizes,
// layout constants and the thermo, reaction and species tables they read.
std::string generate_row_source(const MechanismData& m, const RowLayout& w);

// The launches of a mechanism's wave-cooperative forward kernels.
struct WaveLaunch {
    int block = 64, cells = 1;       // lanes, and cells, of a workgroup
    unsigned lds = 0;                // bytes of a workgroup
    int blocks_per_cu = 1;           // resident workgroups per compute unit
    int64_t blocks(int64_t ncell) const { return (ncell + cells - 1) / cells; }
    int64_t lanes(int64_t ncell) const { return blocks(ncell) * block; }
};

}  // namespace chemmi
