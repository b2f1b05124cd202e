// Internal interface between the C ABI (fv_api.hip) and the kernel launchers.
#pragma once

#include "fv_device.h"

namespace fvk {

// One 2D grid of the fused path (device memory, read uniformly).
// Stage clock record of the batch (per grid and stage, earliest work-item
// start and latest end): each entry is spread over CLK_SLOTS slots, one
// 128-byte line apart, that work items pick by their index, so the per-item
// atomics do not all meet on one address; the slots are folded when the
// step's record is stored.
constexpr int CLK_SLOTS = 16;
constexpr int CLK_PAD = 16;  // unsigned long longs per slot (one 128-byte line)
__host__ __device__ inline int clk_index(int entry, int slot) { return (entry * CLK_SLOTS + slot) * CLK_PAD; }

// Wave-speed maximum of a grid (bit patterns of non-negative doubles), spread
// over slots a 256-byte line apart that waves pick by their work item: device-scope atomics on one address cost about 10 ns each, one after
// the other, and the waves of a stage end together (512^2: 1152 of them made
// the last stage 23.4 us against 11.5 for the one before; over the slots it
// takes 12). The reader takes the maximum of the slots, one per lane.
// Two sets per grid: the stage kernels accumulate in set 0, the wave speed of a
// call's first state goes to set 1; the second stage clears both, so a call
// needs no clearing launch of its own. A grid alone has LAM_SLOTS slots a set,
// the grids of a batch as many as the largest of them needs (lam_slots): every
// wave of stage 1 reads, and each step clears, all of a grid's. 65536 grids of
// 8^2: 1135 us a step with 32 slots each, 1035 with one.
constexpr int LAM_SLOTS = 32;
constexpr int LAM_PAD = 32;  // unsigned long longs per slot (256 bytes)
__host__ __device__ inline int lam_index(int grid, int slots, int slot) { return (2 * grid * slots + slot) * LAM_PAD; }
inline size_t lam_bytes(int ngrids, int slots) { return (size_t)2 * ngrids * slots * LAM_PAD * 8; }
inline unsigned long long* lam_first(unsigned long long* lam) { return lam + lam_index(0, LAM_SLOTS, LAM_SLOTS); }
// A slot per 1024 cells, a power of two.
inline int lam_slots(long long cells) {
    int s = 1;
    while (s < LAM_SLOTS && cells > 1024LL * s) s *= 2;
    return s;
}

// (FGridHead: what the kernels keep in scalar registers.)
struct FGridHead {
    int nx, ny, pitch, strips, work0, scheme;  // scheme: FV_SCHEME_*
    int bcx0, bcx1, bcy0, bcy1, gid, seg;   // gid: the caller's grid index (slots of lam, dt, clocks);
                                            // seg: rows per work item
    long long base;     // element offset of cell (0,0), variable 0
    long long sv;       // per-variable stride
    double ax, ay;      // face areas of x faces (dy) and y faces (dx)
    double inv_vol, inv_dx, inv_dy, cfl, gamma, gm1;
    double mu, kcond, nu_fac;  // viscosity, heat conductivity, max(4/3, gamma / Pr) (viscous variant)
};

struct FGrid : FGridHead {
    double q[2][2][4];  // conserved ghost state of inflow faces per axis and side (the kernels'
                        // boundary variant only: grids with slip walls or inflow faces)
};

// The 3D grid of the fused path (device memory, read uniformly).
struct FGrid3Head {
    int nx, ny, nz, strips, seg, scheme;       // seg: planes per work item
    int bcx0, bcx1, bcy0, bcy1, bcz0, bcz1;
    long long base;                                // element offset of cell (0,0,0), variable 0
    long long sv, py, pz;                          // strides: variable, row (y), plane (z)
    double ax, ay, az;                             // face areas: dy dz, dx dz, dx dy
    double inv_vol, inv_dx, inv_dy, inv_dz, cfl, gamma, gm1;
};

struct FGrid3 : FGrid3Head {
    double q[3][2][5];  // conserved ghost state of inflow faces per axis and side (boundary variant)
};

void launch_bc_fill(double* U, const Geo& g, const BcState& bcs, int gang, int threads, hipStream_t s);
void launch_flux(int ax, const double* U, double* F, const Geo& g, int bx, int threads, hipStream_t s);
void launch_metrics(const double* nodes, double* met, int nx, int ny, hipStream_t s);
void launch_flux_curv(int ax, const double* U, double* F, const Geo& g, const BcState& bcs, int bx, int threads,
                      hipStream_t s);
void launch_visc(int ax, const double* U, double* F, const Geo& g, const BcState& bcs, hipStream_t s);
void launch_residual(const double* Fx, const double* Fy, const double* Fz, const double* S, double* R, const Geo& g,
                     int gang, int threads, hipStream_t s);
// norms[v] = sqrt(sum_e R[v][e]^2 / ncell) with partial (256 * nvar doubles) as scratch.
void launch_residual_norm(const double* R, double* partial, double* norms, const Geo& g, hipStream_t s);
void launch_update(int stage, const double* Un, const double* Us, double* Ud, const double* R, const double* dt,
                   const Geo& g, int gang, int threads, hipStream_t s);
int cfl_blocks(const Geo& g, int gang, int threads);
void launch_cfl(const double* U, double* partial, uint32_t* status, const double* dt_in, double* dt,
                double* dt_out, const Geo& g, int gang, int threads, hipStream_t s);
void launch_set_u32(uint32_t* p, uint32_t v, hipStream_t s);

// fused 2D stages
int fused_items(const FGrid& G, int seg);  // work items of G at segment height seg
int fused_strips(int nx);
void launch_fused_stage(int stage, int waves, const FGrid* grids, int ngrids, int nitems, const double* Un,
                        const double* Us, double* Ud, unsigned long long* lam, double* dtg, const double* dt_fixed,
                        double* dt_out, uint32_t* status, unsigned long long* clk, hipStream_t s,
                        const double* src = nullptr, int mode = 0, const double* met = nullptr,
                        int slots = LAM_SLOTS);
void launch_lam_reset(unsigned long long* lam, int ngrids, int slots, hipStream_t s);
void launch_fused_init(const FGrid* grids, int ngrids, int nitems, const double* U, unsigned long long* lam,
                       uint32_t* status, hipStream_t s, const double* met = nullptr, int slots = LAM_SLOTS);
int fused_slots();
int fused3d_items(const FGrid3& G, int seg);
void launch_fused3d_stage(int stage, int waves, const FGrid3* grid, int nitems, const double* Un, const double* Us,
                          double* Ud, unsigned long long* lam, double* dtg, const double* dt_fixed, double* dt_out,
                          uint32_t* status, hipStream_t s, const double* src = nullptr, double vol = 0.0,
                          bool walls = false);
void launch_fused3d_init(const FGrid3* grid, int nitems, const double* U, unsigned long long* lam,
                         uint32_t* status, hipStream_t s);
int fused3d_slots();
int fused3d_init_items(const FGrid3& G);
int fused3d_auto_seg(const FGrid3& G, int cus);
int fused3d_planes(const FGrid3& G, int seg, int cus);
int fused_auto_seg(const FGrid* grids, int ngrids, int slots);
int fused_rows(const FGrid* grids, int ngrids, int seg, int cus, int per_simd);

// whole 2D steps in one launch each (fv_step2d.hip); cus: the device's compute units. ws: step2d_bytes() of
// scratch; step: the step's number in the call; launch_step2d_init: the first
// step's wave speeds (with dt_in null)
size_t step2d_bytes();
void launch_step2d_init(const FGrid& G, const double* U, double* ws, uint32_t* status, const double* met,
                        hipStream_t s);
bool step2d_pays(const FGrid& G, int cus);
void launch_step2d(const FGrid& G, int cus, const double* gq, const double* Un, double* Ud, double* ws, int step,
                   const double* dt_in, double* dtg, double* dt_out, uint32_t* status, const double* src, int mode,
                   const double* met, hipStream_t s);
void launch_step2d_copy(const FGrid& G, const double* from, double* to, hipStream_t s);

// adjoint: one reverse Runge-Kutta stage (mode 3, 2, 1 for stages 3, 2, 1)
void launch_adj_stage(int mode, const double* Us, const double* w, double* lam, double* lamA, double* lamB, double* R,
                      const double* dt, const Geo& g, const BcState& bcs, hipStream_t s);

}  // namespace fvk
