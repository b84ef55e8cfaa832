// gks_adjoint.h -- discrete adjoint of the S2O4 step with the actuator-line body force (internal).
//
// The reverse sweep linearises the step exactly; the WENO nonlinear weights are either held at their
// forward values (frozen, the default) or differentiated too (exact). Per face direction and stage
// operator the transpose is computed without atomics, every sum in a fixed order: tile by tile the forward
// face pipeline, the reverse of the flux at the Gauss points from the flux seeds and the transposes of the
// t2, t1 and normal reconstructions, down to the adjoints of the cells of the tile's columns; then the sum of
// the tiles' shares. The coefficients of the WENO evaluations (frozen: the weights; exact: the Jacobian row)
// are rebuilt from the values the evaluations read; then the transpose of the ghost-cell fill folds ghost
// adjoints into interior cells.
#pragma once

#include <stddef.h>

#include "gks_body.h"
#include "gks_internal.h"

namespace gks {

// Tile: 16 x 8 faces, four lanes per face, one workgroup per CU (its LDS: 162 KB), two waves per SIMD.
struct AdjTile {
    static constexpr int T2 = 8, THREADS = 64 * T2;
};
constexpr int ADJ_SLOTS = 256;  // workgroups at once (256 CUs); fixed, since the workspace's size depends on the split

// Work split of one direction: marches of `chunk` faces, nch per tile. x1, x2: columns of a tile that the slab
// keeps, 20 x 12, or of a single narrow tile only those the domain's cells reach.
struct AdjSplit {
    int tiles_t1, tiles_t2, chunk, nch, x1, x2;
};
AdjSplit adj_split(int n_n, int n_t1, int n_t2);

enum { ADJ_SUM_ACC, ADJ_SUM_ZERO, ADJ_SUM_LAM_STAR };

struct AdjFaceArgs {
    const double* q[4];     // field in LOCAL variable order (padded)
    // the flux seeds are l[0] lam + l[1] star (of L, stage 1 only) and lt[0] lam + lt[1] star (of L_t); star in
    // stage 1 only. lam, star: padded, local order; seed_lam, seed_star: the same in q's layout
    const double* lam[4];
    const double* star[4];
    const double* seed_lam[4];
    const double* seed_star[4];
    double l[2], lt[2];
    double* slab;           // [tile][march][cell, chunk + 5][variable][x2 t2 rows][x1 t1 columns]: cell adjoints
    double* acc[4];         // padded cell adjoint (LOCAL order), ghost cells zero beforehand
    int sum;                // what adj_sum_kernel adds the direction's cell adjoints to
    int n_n, n_t1, n_t2;
    int tiles_t1, tiles_t2;
    int chunk, nch, n_wg;  // marches of chunk of the n_n + 1 faces, nch per tile, one per workgroup
    int x1, x2;
    long long st_n, st_t1, st_t2;
    long long pad0;
    long long qst_n, qst_t1, qst_t2, qpad0;  // of q and the seeds (the x direction reads [x][z][y] copies)
    // inverse spacings (device, the forward's arrays; 1/h on a uniform axis): normal face spacings
    // [n_n + 1], normal widths [n_n], t1 widths [n_t1], t2 widths [n_t2]
    const double* ihf;
    const double* ihc;
    const double* ih1;
    const double* ih2;
    double eps;
    FluxConst<double> fc;
    int exact;              // 1: the WENO weights are differentiated (Jacobian rows), 0: frozen
};

size_t adjoint_workspace_bytes(int nx, int ny, int nz, int n_act);

struct AdjBuffers {
    double* lam[4];      // padded: adjoint of Q^{n+1}, after the actuator line of Q^{n+1,pre}
    double* lam_star[4]; // padded: adjoint of Q*
    double* lam_new[4];  // padded: adjoint of Q^n, the next step's lam
    double* star_t[4];   // [x][z][y] copy of lam_star, read by the x direction
    double* slab;
    double* pt;          // per-point scratch of the ALM adjoint: [16][n_act]
};

void adjoint_carve(char* base, int nx, int ny, int nz, int n_act, AdjBuffers* b, size_t* total);

hipError_t launch_adj_direction(const AdjFaceArgs& a, int stage, hipStream_t s);
// transpose of the axis-by-axis ghost fill (z, y, x); inflow sides are linearised at the padded field q
// (global variable order) the fill was applied to
hipError_t launch_adj_fold(double* f[4], const GridDesc& g, const int bc[6], const double* const q[4],
                           const double u_in[3], double c, double rho_ref, hipStream_t s);
// interior cells of a padded field, four variables back to back
hipError_t launch_interior(double* dst, const double* const src[4], const GridDesc& g, hipStream_t s);
// the [x][z][y] copy of a padded field
hipError_t launch_adj_transpose(double* const dst[4], const double* const src[4], const GridDesc& g, hipStream_t s);
hipError_t launch_zero(double* y, long long n, hipStream_t s);

// immersed-body adjoint (a body at rest): lam (padded, adjoint of the field after the forcing) becomes
// the adjoint of the field before it, in place
hipError_t launch_ibm_adjoint(double* lam[4], const IbmArgs& a, hipStream_t s);

// actuator-line adjoint
struct AlmAdjArgs {
    AlmArgs fwd;             // forward arguments (positions and per-point data of this step)
    double* lam[4];          // padded adjoint of the field after the projection, then of the one before it
    const double* qpre[4];   // padded field before the projection (FP64)
    double* grad_s;          // n_act, accumulated
    double* pt;              // scratch [16][n_act]
    double w0, w1, inv_n;    // objective weights and 1/(window steps)
};
hipError_t launch_alm_adjoint(const AlmAdjArgs& a, hipStream_t s);

}  // namespace gks
