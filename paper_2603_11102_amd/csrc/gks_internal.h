// gks_internal.h -- structures shared by the host library and the kernels (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gks_device.h"

namespace gks {

constexpr int NG = 3;                    // ghost layers per side
constexpr int TILE1 = 16, TILE2 = 16;    // tangential faces per workgroup (t1 x t2)
constexpr int EXT1 = TILE1 + 4, EXT2 = TILE2 + 4;
constexpr int FACE_THREADS = 512;        // 8 wave64 per workgroup

// Tiles of the order-5 face kernels, TILE1 x T2 faces. FP32: 16 x 16 faces, 512 threads (two waves per
// SIMD, up to 256 registers each), two lanes per face. FP64: four lanes per face, 16 x 12 faces on 768
// threads or 16 x 8 on 512. A step of the 12-row tile takes about 1.3 times a step of the 8-row one for 1.5 times
// the faces, so it wins where both fill the chip and loses on small or badly divided planes (us a step,
// 12 rows / 8 rows: 192 x 96 x 96 channel 1387 / 1508, periodic cubes 128^3 1674 / 1720, 56^3 204 / 226,
// 64^3 281 / 258, 24^3 61 / 54). 16 rows do not fit: 128 registers a thread spill (192 x 96 x 96: 1690 to 1960).
constexpr int FACE64_ROWS[2] = {12, 8};
constexpr double FACE64_STEP[2] = {6000.0, 4600.0};  // ns a face step
constexpr double FACE32_STEP = 4300.0;
// ns: what a face launch costs beyond its face steps, a combine launch, and the latter's time per cell.
// Measured on periodic cubes, us a step, two launches a stage against one and the combine: FP32 16^3 65 / 44,
// 40^3 96 / 84, 56^3 148 / 147, 128^3 906 / 1083; FP64 16^3 62 / 44, 40^3 119 / 110, 128^3 1671 / 1917.
constexpr double FACE_LAUNCH = 1000.0, COMBINE_LAUNCH = 3000.0, COMBINE_CELL32 = 0.039, COMBINE_CELL64 = 0.052;

// Local index (the pass's variable order: density, normal momentum, t1, t2 momenta) of each global
// variable (density, x, y, z momenta) for the x (MODE 3), y (MODE 0) and z (MODE 4) passes.
template <int MODE>
struct LocalOrder;
template <>
struct LocalOrder<3> {
    static constexpr int v[4] = {0, 1, 2, 3};
};
template <>
struct LocalOrder<0> {
    static constexpr int v[4] = {0, 2, 1, 3};
};
template <>
struct LocalOrder<4> {
    static constexpr int v[4] = {0, 2, 3, 1};
};
template <>
struct LocalOrder<5> : LocalOrder<4> {};  // the z pass that leaves its residual to combine_kernel

__host__ __device__ inline int pad8(int n) { return (n + 7) / 8 * 8; }

// Device-resident scalars of a context (lives in the workspace).
constexpr int UMAX_BLOCKS = 2048;  // workgroups of umax_kernel at most, and the room for partial maxima

struct DevState {
    double t, dt, t_next;
    long long step;
    double thrust, torque, power, cp, ct;
    double ibm_force[3];
    unsigned long long ibm_res_bits;
    double win_p, win_t;
    long long win_n;
    double mass, mom[3];
    unsigned long long umax_diag_bits;
    int nonfinite;
    int ibm_iters_used;
    int ibm_outside;  // a moving body's point support left the interior (sticky until new points)
};

// The time step's inputs (cfl <= 0: dt_fixed): partial maxima of |U|^2 and constants.
struct DtArgs {
    DevState* st;
    const double* part;
    int nparts;
    double cfl, hmin, c, dt_fixed;
};
constexpr int DT_THREADS = 512;

// dt = CFL h_min / (|U|_max + C) from the partial maxima, by one workgroup of N threads (max is order
// independent, so the result is deterministic); red: N / 64 doubles of LDS.
template <int N>
__device__ __forceinline__ void dt_update(const DtArgs& a, double* red) {
    double mx = 0.0;
    if (a.cfl > 0.0)
        for (int i = threadIdx.x; i < a.nparts; i += 8 * N) {  // eight loads in flight
            double x[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) x[r] = a.part[min(i + r * N, a.nparts - 1)];
#pragma unroll
            for (int r = 0; r < 8; ++r) mx = fmax(mx, x[r]);
        }
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < N / 64; ++w) mx = fmax(mx, red[w]);
    const double dt = a.cfl > 0.0 ? a.cfl * a.hmin / (sqrt(mx) + a.c) : a.dt_fixed;
    a.st->dt = dt;
    a.st->t_next = a.st->t + dt;
    a.st->ibm_res_bits = 0ULL;
}

// Bookkeeping at the end of a step, by one thread: where no rotor or body follows the stage update, by that kernel.
__device__ __forceinline__ void finish_step(DevState* st) {
    st->t = st->t_next;
    st->step += 1;
    st->win_n += 1;
}

// Arguments of the per-direction face kernel. Arrays are in the face's LOCAL variable order
// (rho', m_normal, m_t1, m_t2); the caller permutes the global pointers. Aligned to 16 bytes, which keeps the second and
// third of a launch's blocks on the boundaries of wide scalar loads (24 x 20 x 18 FP32 step 45.5 us with 8, 45.1 with 16).
template <typename real>
struct alignas(16) FaceArgs {
    const real* q[4];        // reconstructed field (padded layout)
    // residual contributions, four variables per cell in the global order (rho', rho U, rho V, rho W):
    real* r0;                // y pass: L (stage 1), interior layout [cell][4]
    real* r1;                // y pass: L_t, same layout
    real* rx0;               // x pass: L in the blocked layout [z][y/16][x][y%16][4]
    real* rx1;               // x pass: L_t, same layout
    int rx_nx, rx_nyb;       // nx and ceil(ny / 16) of the blocked layout
    real* out_a[4];          // epilogue: stage 1 -> Q*, stage 2 -> Q^{n+1} (padded)
    real* out_b[4];          // epilogue: stage 1 -> S (padded)
    const real* s_in[4];     // epilogue: stage 2 reads S (padded)
    const real* q_c[4];      // epilogue: stage 1 reads Q^n at the cell (padded)
    // FP32 compensated state, interior layout [cell][4] in the global order: the low-order parts of the
    // stage input of the epilogue (Q^n in stage 1, S in stage 2) and of its outputs (Q* and S; Q^{n+1});
    // null in FP64
    const real* lo_in;
    real* lo_a;
    real* lo_b;
    int n_n, n_t1, n_t2;     // interior cells along normal, t1, t2
    int chunk, tiles_t1, tiles_t2;
    int t2;                  // t2 rows of a tile
    // work split of the order-5 face kernel over its n_wg logical workgroups: seg_len == 0, workgroup b
    // marches chunk b / (tiles) of tile b % (tiles); seg_len > 0, it marches cells
    // [b seg_len, (b + 1) seg_len) of the tile-major (tile, cell) order, one segment per tile it meets
    int seg_len, n_wg;
    long long st_n, st_t1, st_t2;     // padded strides
    long long ist_n, ist_t1, ist_t2;  // interior strides
    long long pad0;                   // padded offset of interior cell (0,0,0)
    real inv_hn, inv_h1, inv_h2;
    // inverse spacings (device) of a stretched mesh (stretched != 0): normal face spacings [n_n + 1],
    // normal widths [n_n], t1 widths [n_t1], t2 widths [n_t2]; on a uniform axis every entry is 1/h
    int stretched;
    const real* ihf;
    const real* ihc;
    const real* ih1;
    const real* ih2;
    real eps;
    FluxConst<real> fc;
    real g_global[3];                 // constant body force (x, y, z) for the stage-2 epilogue
    const double* dt_ptr;             // device dt of the current step
    DevState* finish;                 // not null: this launch ends the step (finish_step)
};

// Arguments of the second-order stage kernel; arrays in the global variable order.
template <typename real>
struct Face2Args {
    const real* q[4];     // stage input (padded)
    const real* q_c[4];   // stage 1: Q^n at the cell
    const real* s_in[4];  // stage 2: S
    real* out_a[4];       // stage 1 -> Q*, stage 2 -> Q^{n+1} (padded)
    real* out_b[4];       // stage 1 -> S
    const real* lo_in;    // FP32 compensated state, as in FaceArgs
    real* lo_a;
    real* lo_b;
    int n[3];
    int chunk, tiles_x, tiles_y;
    long long st[3], pad0;
    real inv_h[3];
    int stretched;        // inverse spacings per axis (faces, widths) of a stretched mesh
    const real* ihf[3];
    const real* ihc[3];
    FluxConst<real> fc;
    real g_global[3];
    const double* dt_ptr;
    DevState* finish;     // not null: this launch ends the step (finish_step)
};

// Index of cell (x, y, z) in the blocked layout [z][y/16][x][y%16]: the x pass stores 16 consecutive y
// per row (its lanes run along y), the z pass reads a 16 x 16 (x, y) tile as one contiguous block.
__host__ __device__ inline long long rx_block_index(int x, int y, int z, int nx, int nyb) {
    return (((long long)z * nyb + (y >> 4)) * nx + x) * 16 + (y & 15);
}

struct GridDesc {
    int n[3];                 // interior cells x, y, z
    long long st[3];          // padded strides x, y, z
    long long pad0;           // padded offset of interior cell (0,0,0)
    long long n_padded;       // elements per padded field
    double h[3];              // mean cell size lx/nx, ... (the cell size of a uniform axis)
    double x0[3];
    const double* wrel[3];    // device, n[a]: cell width / h[a] of a stretched axis, null when uniform
};

template <typename real>
struct Field4 {
    real* v[4];
};

// host launchers (gks_stage.hip: FP32 and the work split; gks_stage64.hip: FP64)
template <typename real>
hipError_t launch_face_xy(const FaceArgs<real>& ax, const FaceArgs<real>& ay, int stage, hipStream_t s);
template <typename real>
hipError_t launch_face_z(const FaceArgs<real>& a, int stage, hipStream_t s);
template <typename real>
hipError_t launch_face_xyz(const FaceArgs<real>& ax, const FaceArgs<real>& ay, const FaceArgs<real>& az,
                           const DtArgs& dt, int stage, hipStream_t s);
// resident workgroups of the order-5 face kernels with tiles of t2 rows
template <typename real>
int face_slots(int t2);
#define GKS_FACE_DECL(real)                                                                                     \
    template <>                                                                                                 \
    hipError_t launch_face_xy<real>(const FaceArgs<real>& ax, const FaceArgs<real>& ay, int stage, hipStream_t s); \
    template <>                                                                                                 \
    hipError_t launch_face_z<real>(const FaceArgs<real>& a, int stage, hipStream_t s);                          \
    template <>                                                                                                 \
    hipError_t launch_face_xyz<real>(const FaceArgs<real>& ax, const FaceArgs<real>& ay, const FaceArgs<real>& az, \
                                     const DtArgs& dt, int stage, hipStream_t s);                               \
    template <>                                                                                                 \
    int face_slots<real>(int t2);
GKS_FACE_DECL(float)
GKS_FACE_DECL(double)
#undef GKS_FACE_DECL
// chunk of the launches whose workgroups march aligned chunks (second-order pass, adjoint recompute)
int face_chunk(int n_n, int tiles, int slots);
// Work split of one order-5 launch over the directions that share it: n cells along the normal and tiles per
// direction in, FaceArgs chunk, seg_len, n_wg out; returns the longest workgroup's face steps.
struct FaceDir {
    int n, tiles;
};
struct FaceSplit {
    int chunk, seg_len;
    long long n_wg;
};
int face_split(const FaceDir* dirs, int ndirs, int slots, FaceSplit* out);
// Tiles, work split and launches of a grid's order-5 face passes.
struct FacePlan {
    int side_by_side;  // the three directions of a stage run in one launch
    int rows;          // t2 rows of a tile (FP64: see FACE64_ROWS)
    int chunk[3], seg_len[3], n_wg[3];  // FaceArgs, per direction
};
// slots: workgroups that run at once with tiles of each height (FP32: the first)
FacePlan face_plan(const int n[3], bool f64, const int slots[2]);
// second-order variant (gks_stage2.hip): one launch per stage; stage2_chunk: planes per workgroup
template <typename real>
hipError_t launch_stage2(const Face2Args<real>& a, int stage, hipStream_t s);
int stage2_chunk(const int n[3], int f64);

// host launchers (gks_aux.hip)
template <typename real>
hipError_t launch_ghost(Field4<real> f, const GridDesc& g, int axis, int bc_lo, int bc_hi, const double u_in[3],
                        double c, double rho_ref, hipStream_t s);
// stage update of an order-5 stage whose z pass left its residual in the output fields (launch_face_xyz):
// az: the z pass's arguments
template <typename real>
hipError_t launch_combine(const FaceArgs<real>& az, const GridDesc& g, int stage, hipStream_t s);
template <typename real>
hipError_t launch_umax(Field4<real> f, const GridDesc& g, double rho_ref, double* part, hipStream_t s);
// workgroups of ghost_transpose_kernel (one partial maximum each) and of umax_kernel
int ghost_parts(const int n[3]);
int umax_parts(const int n[3]);
hipError_t launch_zero_words(void* p, size_t bytes, hipStream_t s);
template <typename real>
hipError_t launch_ghost_shell(Field4<real> q, const GridDesc& gd, const int bc[6], const double u_in[3], double c,
                              double rho_ref, hipStream_t s);
template <typename real>
hipError_t launch_ghost_transpose(Field4<real> q, Field4<real> qt, const GridDesc& gd, const int bc[6],
                                  const double u_in[3], double c, double rho_ref, double* part, hipStream_t s);
hipError_t launch_dt(const DtArgs& a, hipStream_t s);
hipError_t launch_finish(DevState* st, int has_rotor, double* hist, hipStream_t s);
hipError_t launch_window_reset(DevState* st, hipStream_t s);
template <typename real>
hipError_t launch_diag(Field4<real> f, const real* lo, const GridDesc& g, double rho_ref, double* partials, int nblk,
                       DevState* st,
                       hipStream_t s);
int diag_blocks(const GridDesc& g);
// checkpointed interior to q with its ghost cells and to the [x][z][y] copy; t (or null): the step's time
hipError_t launch_restore(const double* const from[4], Field4<double> q, Field4<double> qt, const GridDesc& gd,
                          const int bc[6], const double u_in[3], double c, double rho_ref, const double* t,
                          const DtArgs& dt, hipStream_t s);
hipError_t launch_copy_field(const void* src, void* dst, size_t bytes, hipStream_t s);

}  // namespace gks
