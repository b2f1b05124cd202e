// A whole SSP-RK3 step of a 2D grid in one launch, for grids whose step is
// bound by launches and latency (FP64, gfx950).
//
// A workgroup owns a tile of TX x TY cells. It loads the tile and six cells
// around it into LDS and runs the three Runge-Kutta stages there: stage 1 on
// the tile and four cells around it, stage 2 on two, stage 3 on the tile. The
// cells around a tile are computed again by its neighbours, so no tile waits
// for another one: a step needs one launch instead of three, each of which
// took 6-7 us of launch, table reads and a serial march over its rows however
// small the grid (the times stand at launch_step2d_m). The price is 1.6 times
// the face evaluations at 16 x 16.
//
// In a stage the x and y faces are handed out to the waves in runs of 64, one
// face per lane, and their fluxes go to LDS; then each cell takes its four
// fluxes and the stage combination. Ghost cells: the load maps positions
// outside the grid through the boundary kinds; periodic halos then advance
// like any other cell, and behind the other kinds the two ghost layers are
// filled again from the tile after each stage.
//
// The step reads U^n from one buffer and writes U^{n+1} to another one (its
// neighbours still read U^n). The wave-speed maximum of U^{n+1} goes to one of
// three slot sets in turn: a step reads the set of the step before, adds to
// its own and clears the next one's.
//
// The arithmetic of a face and a cell is that of the stage kernels
// (fv_fused2d.h), operation for operation: the same bits.
#include "fv_fused2d.h"

namespace fvk {

constexpr int SHALO = 6;

template <int TX, int TY, int T, int MODE>
struct StepLds {
    static constexpr int RX = TX + 2 * SHALO, RY = TY + 2 * SHALO;
    double A[4][RX * RY];               // state of the stage, [v][hy][hx]
    double FX[4][(TX + 9) * (TY + 8)];  // x-face fluxes (times 2; curvilinear: times the length)
    double FY[4][(TX + 8) * (TY + 9)];  // y-face fluxes
    double W[MODE == 2 ? 3 : 1][MODE == 2 ? (TX + 10) * (TY + 10) : 1];  // viscous: u, v, T within five cells
    int mx[RX], my[RY];                 // cell read at a position
    int kx[RX], ky[RY];                 // ghost rule: 0 none, 2 kind + side for a wall (2) or an inflow face (3)
    double lmax[T / 64];
    uint32_t fl[T / 64];
};

// Cell read at position p of an axis of n cells, any number of periods or
// cells outside it (only two of them matter behind the other kinds).
__device__ __forceinline__ int step_map(int p, int n, int lo, int hi) {
    if (p >= 0 && p < n) return p;
    if (lo == 0) {
        while (p < 0) p += n;  // once, but on the smallest grids
        while (p >= n) p -= n;
        return p;
    }
    const int kind = p < 0 ? lo : hi;
    if (kind == 2 && p >= -2 && p <= n + 1) return p < 0 ? -1 - p : 2 * n - 1 - p;
    return p < 0 ? 0 : n - 1;
}

__device__ __forceinline__ int step_rule(int p, int n, int lo, int hi) {
    if (p >= 0 && p < n) return 0;
    const int kind = p < 0 ? lo : hi;
    return kind >= 2 ? 2 * kind + (p < 0 ? 0 : 1) : 0;
}

// What the stages of a tile share.
struct StepArgs {
    const double *Un, *src, *met, *gq;
    double* Ud;
    double s;    // -dt / |Omega| (curvilinear: -dt)
    int tx0, ty0;
    bool edge;   // the tile reads ghost cells that are filled after each stage
};

// Applies the ghost rules kx, ky of a position to the cell it reads (y first,
// then x, as in the stage kernels); (mx, my): the cell read.
template <int MODE>
__device__ __forceinline__ void step_ghost(const FGridHead& G, const StepArgs& a, int kx, int ky, int mx, int my,
                                           double* w) {
    if (ky >= 6) {
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = a.gq[(2 + (ky & 1)) * 4 + v];
    } else if (ky >= 4) {
        if (MODE == 3) {
            const MetricOffsets mo = metric_offsets(G.nx, G.ny);
            const long long f = mo.fy + (long long)((ky & 1) ? G.ny : 0) * G.nx + mx;
            const double nx = a.met[f], ny = a.met[f + mo.nfy];
            const double mn = w[1] * nx + w[2] * ny;
            w[1] -= 2.0 * mn * nx;
            w[2] -= 2.0 * mn * ny;
        } else {
            w[2] = -w[2];
        }
    }
    if (kx >= 6) {
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = a.gq[(kx & 1) * 4 + v];
    } else if (kx >= 4) {
        if (MODE == 3) {
            const MetricOffsets mo = metric_offsets(G.nx, G.ny);
            const long long f = mo.fx + (long long)my * (G.nx + 1) + ((kx & 1) ? G.nx : 0);
            const double nx = a.met[f], ny = a.met[f + mo.nfx];
            const double mn = w[1] * nx + w[2] * ny;
            const double m1 = w[1] - 2.0 * mn * nx, m2 = w[2] - 2.0 * mn * ny;
            w[1] = m1;
            w[2] = m2;
        } else {
            w[1] = -w[1];
        }
    }
}

// Unit normal and length of a face: f its index in its block.
__device__ __forceinline__ void step_face(const double* met, long long base, long long stride, long long f,
                                          double* m) {
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k] = met[base + k * stride + f];
}

template <int LIM>
__device__ __forceinline__ void step_states(double q0, double q1, double q2, double q3, double ka, double kb,
                                            double& qL, double& qR) {
    const double dm = q1 - q0, dc = q2 - q1, dp = q3 - q2;
    if (LIM == 2) {
        muscl_kappa_diffs(q1, q2, dm, dc, dp, ka, kb, qL, qR);
    } else if (LIM == 1) {
        qL = q1 + 0.5 * dm;
        qR = q2 - 0.5 * dp;
    } else {
        qL = q1 + 0.5 * limited_slope<LIM>(dm, dc);
        qR = q2 - 0.5 * limited_slope<LIM>(dc, dp);
    }
}

template <int TX, int TY, int T, int STAGE, int LIM, bool SRC, int MODE>
__device__ __forceinline__ void step_stage(const FGridHead& G, StepLds<TX, TY, T, MODE>& L, const StepArgs& a,
                                           double ka, double kb, double& lmax, uint32_t& fl) {
    constexpr int h = 4 - 2 * STAGE;               // cells around the tile that the stage computes
    constexpr int RX = TX + 2 * SHALO;
    constexpr int CW = TX + 2 * h, CH = TY + 2 * h, NC = CW * CH;
    constexpr int XW = CW + 1, NXF = XW * CH, NYF = CW * (CH + 1);
    constexpr int XC = (NXF + 63) / 64, YC = (NYF + 63) / 64;
    constexpr int O = SHALO - h;                   // region position of the stage's first cell
    constexpr int WX = TX + 10;                    // viscous: W holds region positions 1 .. RX - 2
    constexpr bool VISC = MODE == 2, CURV = MODE == 3;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const double hax = 0.5 * G.ax, hay = 0.5 * G.ay;
    const MetricOffsets mo = metric_offsets(G.nx, G.ny);
    if (VISC) {
#pragma clang fp contract(on)
        constexpr int VW = CW + 2, NV = VW * (CH + 2);  // the stage's cells and one around them
        for (int c = tid; c < NV; c += T) {
            const int hy = O - 1 + c / VW, hx = O - 1 + c % VW, e = hy * RX + hx;
            const double q[4] = {L.A[0][e], L.A[1][e], L.A[2][e], L.A[3][e]};
            double w[3];
            visc_w2(q, G.gm1, w);
#pragma unroll
            for (int m = 0; m < 3; ++m) L.W[m][(hy - 1) * WX + hx - 1] = w[m];
        }
        __syncthreads();
    }
    // U^n of this thread's first cell, requested ahead of the fluxes
    auto cell_offset = [&](int c) {
        return (uint32_t)(L.my[O + c / CW] * G.pitch + L.mx[O + c % CW]) * 8u;
    };
    const Rsrc rn = grid_rsrc(a.Un + G.base, 4 * G.sv * 8);
    const uint32_t vstride = (uint32_t)(G.sv * 8);
    double un[4];
    if (STAGE > 0) {
        const uint32_t o = cell_offset(tid < NC ? tid : 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) un[v] = ld_buf(rn, o, v * vstride);
    }
    for (int t = wave; t < XC + YC; t += T / 64) {
        double qL[4], qR[4], F[4];
        if (t < XC) {
            // x face between cells fx - 1 and fx of row fy (lanes past the last face repeat it)
            const int f0 = t * 64 + lane, f = f0 < NXF ? f0 : NXF - 1;
            const int fy = f / XW, fx = f - fy * XW;
            const int e = (O + fy) * RX + O + fx - 2;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                step_states<LIM>(L.A[v][e], L.A[v][e + 1], L.A[v][e + 2], L.A[v][e + 3], ka, kb, qL[v], qR[v]);
            if (CURV) {
                int gx = a.tx0 - h + fx, gy = a.ty0 - h + fy;
                gx = gx < 0 ? 0 : (gx > G.nx ? G.nx : gx);
                gy = gy < 0 ? 0 : (gy > G.ny - 1 ? G.ny - 1 : gy);
                double m[3];
                step_face(a.met, mo.fx, mo.nfx, (long long)gy * (G.nx + 1) + gx, m);
                roe_flux_n2(qL, qR, m[0], m[1], G.gm1, F);
#pragma unroll
                for (int v = 0; v < 4; ++v) F[v] *= m[2];
            } else {
                roe_flux<2, 0, true>(qL, qR, G.gm1, F);
            }
            if (VISC) {
#pragma clang fp contract(on)
                const int w0 = (O + fy - 1) * WX + O + fx - 2;  // W of cell fx - 1
                double wl[3], wr[3], dt[3], V[3];
                const double qdy = 0.25 * G.inv_dy;
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    wl[m] = L.W[m][w0];
                    wr[m] = L.W[m][w0 + 1];
                    dt[m] = ((L.W[m][w0 + WX] - L.W[m][w0 - WX]) + (L.W[m][w0 + 1 + WX] - L.W[m][w0 + 1 - WX])) * qdy;
                }
                visc_flux2<0>(wl, wr, dt, G.inv_dx, G.mu, G.kcond, V);
#pragma unroll
                for (int m = 0; m < 3; ++m) F[1 + m] = fma(-2.0, V[m], F[1 + m]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) L.FX[v][f] = F[v];
        } else {
            // y face between rows fy - 1 and fy of column fx
            const int f0 = (t - XC) * 64 + lane, f = f0 < NYF ? f0 : NYF - 1;
            const int fy = f / CW, fx = f - fy * CW;
            const int e = (O + fy - 2) * RX + O + fx;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                step_states<LIM>(L.A[v][e], L.A[v][e + RX], L.A[v][e + 2 * RX], L.A[v][e + 3 * RX], ka, kb, qL[v],
                                 qR[v]);
            if (CURV) {
                int gx = a.tx0 - h + fx, gy = a.ty0 - h + fy;
                gx = gx < 0 ? 0 : (gx > G.nx - 1 ? G.nx - 1 : gx);
                gy = gy < 0 ? 0 : (gy > G.ny ? G.ny : gy);
                double m[3];
                step_face(a.met, mo.fy, mo.nfy, (long long)gy * G.nx + gx, m);
                roe_flux_n2(qL, qR, m[0], m[1], G.gm1, F);
#pragma unroll
                for (int v = 0; v < 4; ++v) F[v] *= m[2];
            } else {
                roe_flux<2, 1, true>(qL, qR, G.gm1, F);
            }
            if (VISC) {
#pragma clang fp contract(on)
                const int w0 = (O + fy - 2) * WX + O + fx - 1;  // W of row fy - 1
                double wl[3], wr[3], dt[3], V[3];
                const double qdx = 0.25 * G.inv_dx;
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    wl[m] = L.W[m][w0];
                    wr[m] = L.W[m][w0 + WX];
                    dt[m] = ((L.W[m][w0 + 1] - L.W[m][w0 - 1]) + (L.W[m][w0 + WX + 1] - L.W[m][w0 + WX - 1])) * qdx;
                }
                visc_flux2<1>(wl, wr, dt, G.inv_dy, G.mu, G.kcond, V);
#pragma unroll
                for (int m = 0; m < 3; ++m) F[1 + m] = fma(-2.0, V[m], F[1 + m]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) L.FY[v][f] = F[v];
        }
    }
    __syncthreads();
    const double vol = G.ax * G.ay;
    for (int c = tid; c < NC; c += T) {
        const int cy = c / CW, cx = c - cy * CW;
        const int e = (O + cy) * RX + O + cx;
        const int fx = cy * XW + cx;
        const int gx = a.tx0 - h + cx, gy = a.ty0 - h + cy;
        const bool own = STAGE == 2 && gx < G.nx && gy < G.ny;
        long long ce = 0;  // curvilinear: the cell's metric entry
        if (CURV) {
            const int mx = gx < 0 ? 0 : (gx > G.nx - 1 ? G.nx - 1 : gx);
            const int my = gy < 0 ? 0 : (gy > G.ny - 1 ? G.ny - 1 : gy);
            ce = mo.cell + (long long)my * G.nx + mx;
        }
        double Sv[4];
        if (SRC) {
            const long long plane = (long long)G.nx * G.ny;
            const long long p = (long long)L.my[O + cy] * G.nx + L.mx[O + cx];
#pragma unroll
            for (int v = 0; v < 4; ++v) Sv[v] = a.src[v * plane + p];
        }
        if (STAGE > 0 && NC > T && c >= T) {
            const uint32_t o = cell_offset(c);
#pragma unroll
            for (int v = 0; v < 4; ++v) un[v] = ld_buf(rn, o, v * vstride);
        }
        const double sc = CURV ? a.s * a.met[ce + mo.nc] : a.s;
        double out[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double cv = L.A[v][e];
            const double Fxl = L.FX[v][fx], Fxr = L.FX[v][fx + 1], Fyl = L.FY[v][c], Fyr = L.FY[v][c + CW];
            double r = CURV ? Fxr - Fxl : (Fxr - Fxl) * hax;
            if (CURV) r += Fyr - Fyl;
            else r += (Fyr - Fyl) * hay;
            if (SRC) r -= (CURV ? a.met[ce] : vol) * Sv[v];
            if (STAGE == 0) out[v] = cv + sc * r;
            else if (STAGE == 1) out[v] = 0.75 * un[v] + 0.25 * (cv + sc * r);
            else out[v] = (1.0 / 3.0) * un[v] + (2.0 / 3.0) * (cv + sc * r);
        }
        if (STAGE < 2) {
#pragma unroll
            for (int v = 0; v < 4; ++v) L.A[v][e] = out[v];
        } else if (own) {
            const long long p = G.base + (long long)gy * G.pitch + gx;
#pragma unroll
            for (int v = 0; v < 4; ++v) a.Ud[v * G.sv + p] = out[v];
            if (CURV) {
                double xa[3], xb[3], ya[3], yb[3];
                const long long fxi = (long long)gy * (G.nx + 1) + gx, fyi = (long long)gy * G.nx + gx;
                step_face(a.met, mo.fx, mo.nfx, fxi, xa);
                step_face(a.met, mo.fx, mo.nfx, fxi + 1, xb);
                step_face(a.met, mo.fy, mo.nfy, fyi, ya);
                step_face(a.met, mo.fy, mo.nfy, fyi + G.nx, yb);
                lmax = fmax(lmax, curv_cell_lambda(out, G.gamma, G.gm1, xa, xb, ya, yb, a.met[ce], &fl));
            } else {
                const double idx[2] = {G.inv_dx, G.inv_dy};
                double lam = cell_lambda<2>(out, G.gamma, G.gm1, idx, fl);
                if (VISC) lam += 2.0 * ((G.mu / out[0]) * G.nu_fac) * (G.inv_dx * G.inv_dx + G.inv_dy * G.inv_dy);
                lmax = fmax(lmax, lam);
            }
        }
    }
    if (STAGE < 2) {
        __syncthreads();
        if (a.edge) {
            // the two ghost layers behind non-periodic faces, from the stage's
            // cells: within two cells of the next stage's (one in a corner is enough)
            constexpr int GW = CW, NG2 = GW * CH;
            for (int c = tid; c < NG2; c += T) {
                const int hy = O + c / GW, hx = O + c % GW;
                const int gx = a.tx0 - SHALO + hx, gy = a.ty0 - SHALO + hy;
                const bool ox = (gx < 0 && G.bcx0 != 0 && gx >= -2) || (gx >= G.nx && G.bcx1 != 0 && gx < G.nx + 2);
                const bool oy = (gy < 0 && G.bcy0 != 0 && gy >= -2) || (gy >= G.ny && G.bcy1 != 0 && gy < G.ny + 2);
                const bool bx = G.bcx0 != 0 && (gx < -2 || gx >= G.nx + 2), by = G.bcy0 != 0 && (gy < -2 || gy >= G.ny + 2);
                if (!(ox || oy) || bx || by) continue;
                // the cell read, as a position of the region
                const int sx = ox ? L.mx[hx] - a.tx0 + SHALO : hx, sy = oy ? L.my[hy] - a.ty0 + SHALO : hy;
                const int se = sy * RX + sx;
                double w[4] = {L.A[0][se], L.A[1][se], L.A[2][se], L.A[3][se]};
                if (MODE >= 1) step_ghost<MODE>(G, a, ox ? L.kx[hx] : 0, oy ? L.ky[hy] : 0, L.mx[hx], L.my[hy], w);
#pragma unroll
                for (int v = 0; v < 4; ++v) L.A[v][hy * RX + hx] = w[v];
            }
            __syncthreads();
        }
    }
}

template <int TX, int TY, int T, int LIM, bool SRC, int MODE>
__device__ __forceinline__ void step_stages(const FGridHead& G, StepLds<TX, TY, T, MODE>& L, const StepArgs& a,
                                            double ka, double kb, double& lmax, uint32_t& fl) {
    step_stage<TX, TY, T, 0, LIM, SRC, MODE>(G, L, a, ka, kb, lmax, fl);
    step_stage<TX, TY, T, 1, LIM, SRC, MODE>(G, L, a, ka, kb, lmax, fl);
    step_stage<TX, TY, T, 2, LIM, SRC, MODE>(G, L, a, ka, kb, lmax, fl);
}

// lam_in: the wave speeds of U^n, n_in values (null with dt_fixed); lam_out:
// the slots that U^{n+1}'s go to (null: not wanted), lam_clear: the slots that
// the next step adds to. check: raise the flags of U^n too (the first step of
// a call with given step sizes; else the initial wave-speed kernel does).
template <int TX, int TY, int T, bool SRC, int MODE>
__global__ void __launch_bounds__(T) k_step2d(FGridHead G, const double* __restrict__ gq, const double* __restrict__ Un,
                                              double* __restrict__ Ud, const double* __restrict__ lam_in, int n_in,
                                              int stride_in, unsigned long long* lam_out,
                                              unsigned long long* lam_clear_set, const double* __restrict__ dt_fixed,
                                              double* __restrict__ dtg, double* __restrict__ dt_out,
                                              uint32_t* __restrict__ status, const double* __restrict__ src,
                                              const double* __restrict__ met, bool check) {
    __shared__ StepLds<TX, TY, T, MODE> L;
    constexpr int RX = TX + 2 * SHALO, RY = TY + 2 * SHALO, NR = RX * RY, IT = (NR + T - 1) / T;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (G.nx + TX - 1) / TX;
    const int tile = xcd_block(blockIdx.x, gridDim.x);
    StepArgs a;
    a.Un = Un;
    a.Ud = Ud;
    a.src = src;
    a.met = met;
    a.gq = gq;
    a.tx0 = (tile % tiles_x) * TX;
    a.ty0 = (tile / tiles_x) * TY;
    // tiles that read ghost cells behind a non-periodic face (its axis is not periodic on either side)
    a.edge = (G.bcx0 != 0 && (a.tx0 < SHALO || a.tx0 + TX + SHALO > G.nx)) ||
             (G.bcy0 != 0 && (a.ty0 < SHALO || a.ty0 + TY + SHALO > G.ny));
    // the tile and its halo
    const Rsrc rn = grid_rsrc(Un + G.base, 4 * G.sv * 8);
    const uint32_t vstride = (uint32_t)(G.sv * 8);
    double q[IT][4];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int c = tid + k * T < NR ? tid + k * T : NR - 1;
        const int x = step_map(a.tx0 - SHALO + c % RX, G.nx, G.bcx0, G.bcx1);
        const int y = step_map(a.ty0 - SHALO + c / RX, G.ny, G.bcy0, G.bcy1);
        const uint32_t o = (uint32_t)(y * G.pitch + x) * 8u;
#pragma unroll
        for (int v = 0; v < 4; ++v) q[k][v] = ld_buf(rn, o, v * vstride);
    }
    double dt;
    if (dt_fixed) {
        dt = *dt_fixed;
    } else {
        double m = 0.0;
        for (int i = lane; i < n_in; i += 64) m = fmax(m, lam_in[(long long)i * stride_in]);
        dt = G.cfl / wave_max_d(m);
    }
    a.s = from_lane(MODE == 3 ? -dt : -dt * G.inv_vol, 0);
    if (blockIdx.x == 0) {
        if (tid == 0) {
            *dtg = dt;
            if (dt_out) *dt_out = dt;
            if (!(dt > 0.0) || isinf(dt)) atomicOr(status, 8u);
        }
        if (lam_clear_set)
            for (int i = tid; i < LAM_SLOTS; i += T) lam_clear_set[i * LAM_PAD] = 0ull;
    }
    for (int i = tid; i < RX + RY; i += T) {
        if (i < RX) {
            const int p = a.tx0 - SHALO + i;
            L.mx[i] = step_map(p, G.nx, G.bcx0, G.bcx1);
            L.kx[i] = step_rule(p, G.nx, G.bcx0, G.bcx1);
        } else {
            const int p = a.ty0 - SHALO + i - RX;
            L.my[i - RX] = step_map(p, G.ny, G.bcy0, G.bcy1);
            L.ky[i - RX] = step_rule(p, G.ny, G.bcy0, G.bcy1);
        }
    }
    double lmax = 0.0;
    uint32_t fl = 0;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int c = tid + k * T;
        if (c < NR) {
            const int hx = c % RX, hy = c / RX;
            const int gx = a.tx0 - SHALO + hx, gy = a.ty0 - SHALO + hy;
            if (check && hx >= SHALO && hx < SHALO + TX && hy >= SHALO && hy < SHALO + TY && gx < G.nx && gy < G.ny) {
                const double idx[2] = {G.inv_dx, G.inv_dy};
                (void)cell_lambda<2>(q[k], G.gamma, G.gm1, idx, fl);
            }
            if (MODE >= 1 && a.edge) {
                const int kx = step_rule(gx, G.nx, G.bcx0, G.bcx1), ky = step_rule(gy, G.ny, G.bcy0, G.bcy1);
                if (kx | ky)
                    step_ghost<MODE>(G, a, kx, ky, step_map(gx, G.nx, G.bcx0, G.bcx1),
                                     step_map(gy, G.ny, G.bcy0, G.bcy1), q[k]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) L.A[v][c] = q[k][v];
        }
    }
    __syncthreads();
    if (G.scheme == 0) {
        step_stages<TX, TY, T, 0, SRC, MODE>(G, L, a, 0.0, 0.0, lmax, fl);
    } else if (G.scheme == 5) {
        step_stages<TX, TY, T, 3, SRC, MODE>(G, L, a, 0.0, 0.0, lmax, fl);
    } else if (G.scheme == 1) {
        step_stages<TX, TY, T, 1, SRC, MODE>(G, L, a, 0.0, 0.0, lmax, fl);
    } else {
        double ka, kb;
        kappa_weights(G.scheme, ka, kb);
        step_stages<TX, TY, T, 2, SRC, MODE>(G, L, a, ka, kb, lmax, fl);
    }
    lmax = wave_max_d(lmax);
    fl = wave_or(fl);
    if (lane == 0) {
        L.lmax[wave] = lmax;
        L.fl[wave] = fl;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < T / 64; ++w) {
            lmax = fmax(lmax, L.lmax[w]);
            fl |= L.fl[w];
        }
        if (lam_out) lam_add(lam_out, 0, LAM_SLOTS, (int)blockIdx.x, lmax);
        if (fl) atomicOr(status, fl);
    }
}

// lambda_max of U (the first step's dt), one value per workgroup in out, and
// the clearing of the slots the first step adds to.
constexpr int SINIT = 256;  // workgroups
template <bool CURV>
__global__ void __launch_bounds__(256) k_step2d_lambda(FGridHead G, const double* __restrict__ U,
                                                       double* __restrict__ out, unsigned long long* lam_clear_set,
                                                       uint32_t* __restrict__ status, const double* __restrict__ met) {
    __shared__ double sm[4];
    const int tid = threadIdx.x;
    double lmax = 0.0;
    uint32_t fl = 0;
    if (blockIdx.x == 0 && tid < LAM_SLOTS) lam_clear_set[tid * LAM_PAD] = 0ull;
    const uint32_t n = (uint32_t)G.nx * (uint32_t)G.ny, step = gridDim.x * 256u;
    const MetricOffsets mo = metric_offsets(G.nx, G.ny);
    for (uint32_t e0 = blockIdx.x * 256u + tid; e0 < n; e0 += 4 * step) {
        double q[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t e = e0 + k * step < n ? e0 + k * step : e0;
            const uint32_t j = e / (uint32_t)G.nx, i = e - j * (uint32_t)G.nx;
            const long long p = G.base + (long long)j * G.pitch + i;
#pragma unroll
            for (int v = 0; v < 4; ++v) q[k][v] = U[v * G.sv + p];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double idx[2] = {G.inv_dx, G.inv_dy};
            double lam = cell_lambda<2>(q[k], G.gamma, G.gm1, idx, fl);
            if (G.mu > 0.0) lam += 2.0 * ((G.mu / q[k][0]) * G.nu_fac) * (G.inv_dx * G.inv_dx + G.inv_dy * G.inv_dy);
            if (CURV) {
                const uint32_t e = e0 + k * step < n ? e0 + k * step : e0;
                const uint32_t j = e / (uint32_t)G.nx, i = e - j * (uint32_t)G.nx;
                double xa[3], xb[3], ya[3], yb[3];
                const long long fxi = (long long)j * (G.nx + 1) + i;
                step_face(met, mo.fx, mo.nfx, fxi, xa);
                step_face(met, mo.fx, mo.nfx, fxi + 1, xb);
                step_face(met, mo.fy, mo.nfy, (long long)e, ya);
                step_face(met, mo.fy, mo.nfy, (long long)e + G.nx, yb);
                lam = curv_cell_lambda(q[k], G.gamma, G.gm1, xa, xb, ya, yb, met[mo.cell + e]);
            }
            lmax = fmax(lmax, lam);
        }
    }
    lmax = wave_max_d(lmax);
    fl = wave_or(fl);
    if ((tid & 63) == 0) {
        sm[tid >> 6] = lmax;
        if (fl) atomicOr(status, fl);
    }
    __syncthreads();
    if (tid == 0) out[blockIdx.x] = fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]));
}

// The interior of a state (the result of an odd number of steps is in the
// workspace's buffer).
__global__ void __launch_bounds__(256) k_step2d_copy(FGridHead G, const double* __restrict__ from,
                                                     double* __restrict__ to) {
    const uint32_t n = (uint32_t)G.nx * (uint32_t)G.ny;
    for (uint32_t e = blockIdx.x * 256u + threadIdx.x; e < n; e += gridDim.x * 256u) {
        const uint32_t j = e / (uint32_t)G.nx, i = e - j * (uint32_t)G.nx;
        const long long p = G.base + (long long)j * G.pitch + i;
        double q[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) q[v] = from[v * G.sv + p];
#pragma unroll
        for (int v = 0; v < 4; ++v) to[v * G.sv + p] = q[v];
    }
}

// ---------------------------------------------------------------------------

size_t step2d_bytes() { return 8 * (size_t)SINIT + 3 * 8 * (size_t)LAM_SLOTS * LAM_PAD; }

template <int TX, int TY, int T, bool SRC, int MODE>
static void launch_step2d_t(const FGrid& G, const double* gq, const double* Un, double* Ud, double* ws, int step,
                            const double* dt_in, double* dtg, double* dt_out, uint32_t* status, const double* src,
                            const double* met, hipStream_t s) {
    // the three slot sets follow the initial values
    unsigned long long* set = (unsigned long long*)(ws + SINIT);
    constexpr int SET = LAM_SLOTS * LAM_PAD;
    const double* lam_in = step == 0 ? ws : (const double*)(set + ((step + 2) % 3) * SET);
    const int tiles = ((G.nx + TX - 1) / TX) * ((G.ny + TY - 1) / TY);
    hipLaunchKernelGGL((k_step2d<TX, TY, T, SRC, MODE>), dim3(tiles), dim3(T), 0, s, (const FGridHead&)G, gq, Un, Ud,
                       lam_in, step == 0 ? SINIT : LAM_SLOTS, step == 0 ? 1 : LAM_PAD,
                       dt_in ? nullptr : set + (step % 3) * SET, dt_in ? nullptr : set + ((step + 1) % 3) * SET, dt_in,
                       dtg, dt_out, status, src, met, dt_in && step == 0);
}

static inline int step2d_tiles(const FGrid& G, int t) { return ((G.nx + t - 1) / t) * ((G.ny + t - 1) / t); }

// A step in one launch pays while its 16 x 16 tiles are all resident at once,
// two to a CU (their LDS): one more round and the stage kernels, which compute
// no face twice, are as fast (table below).
bool step2d_pays(const FGrid& G, int cus) {
    return (long long)G.nx * G.ny <= 512LL * cus && step2d_tiles(G, 16) <= 2 * cus;
}

template <bool SRC, int MODE>
static void launch_step2d_m(const FGrid& G, int cus, const double* gq, const double* Un, double* Ud, double* ws,
                            int step, const double* dt_in, double* dtg, double* dt_out, uint32_t* status, const double* src,
                            const double* met, hipStream_t s) {
    // the smallest tile that leaves at most one to a CU (its serial part is
    // the shortest), else 16 x 16: us per step of a vortex
    //            8 x 8   12 x 12   16 x 16   stage kernels
    //   64^2      8.0      9.5      10.8         20.2
    //   128^2     9.0      9.9      11.1         20.5
    //   192^2    13.1     10.4      11.1         20.6
    //   256^2    17.4     14.2      11.5         21.1
    //   320^2    26.3     17.9      16.8         21.3
    //   384^2    32.1     22.8      23.4         21.8
    if (step2d_tiles(G, 8) <= cus)
        launch_step2d_t<8, 8, 512, SRC, MODE>(G, gq, Un, Ud, ws, step, dt_in, dtg, dt_out, status, src, met, s);
    else if (step2d_tiles(G, 12) <= cus)
        launch_step2d_t<12, 12, 512, SRC, MODE>(G, gq, Un, Ud, ws, step, dt_in, dtg, dt_out, status, src, met, s);
    else
        launch_step2d_t<16, 16, 512, SRC, MODE>(G, gq, Un, Ud, ws, step, dt_in, dtg, dt_out, status, src, met, s);
}

void launch_step2d_init(const FGrid& G, const double* U, double* ws, uint32_t* status, const double* met,
                        hipStream_t s) {
    unsigned long long* set = (unsigned long long*)(ws + SINIT);
    if (met)
        hipLaunchKernelGGL(k_step2d_lambda<true>, dim3(SINIT), dim3(256), 0, s, (const FGridHead&)G, U, ws, set, status,
                           met);
    else
        hipLaunchKernelGGL(k_step2d_lambda<false>, dim3(SINIT), dim3(256), 0, s, (const FGridHead&)G, U, ws, set,
                           status, met);
}

void launch_step2d(const FGrid& G, int cus, const double* gq, const double* Un, double* Ud, double* ws, int step,
                   const double* dt_in, double* dtg, double* dt_out, uint32_t* status, const double* src, int mode,
                   const double* met, hipStream_t s) {
#define FV_LS(SRCB, M) launch_step2d_m<SRCB, M>(G, cus, gq, Un, Ud, ws, step, dt_in, dtg, dt_out, status, src, met, s)
    if (src) {
        if (mode == 3) FV_LS(true, 3);
        else if (mode == 2) FV_LS(true, 2);
        else if (mode == 1) FV_LS(true, 1);
        else FV_LS(true, 0);
    } else {
        if (mode == 3) FV_LS(false, 3);
        else if (mode == 2) FV_LS(false, 2);
        else if (mode == 1) FV_LS(false, 1);
        else FV_LS(false, 0);
    }
#undef FV_LS
}

void launch_step2d_copy(const FGrid& G, const double* from, double* to, hipStream_t s) {
    const long long n = (long long)G.nx * G.ny;
    const long long blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_step2d_copy, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, s,
                       (const FGridHead&)G, from, to);
}

}  // namespace fvk
