// Adjoint (transpose-Jacobian) of the residual and of the SSP-RK3 stage
// combinations, FP64, gfx950.
//
// One kernel per reverse Runge-Kutta stage. A workgroup owns a tile of cells
// (2D 16 x 12, 3D 16 x 4 x 4) and, axis by axis:
//   1. evaluates the reverse of every face whose stencil holds a cell of the
//      tile (the tile's faces along the axis and three more): the MUSCL face
//      states from the four stencil cells (ghost positions mapped by the face
//      kinds: periodic wrap, transmissive clamp, the mirror cell with the
//      normal momentum reversed behind a slip wall, the given state behind an
//      inflow face), the reverse of the Roe flux with the face adjoint
//      Fb = area (w_left - w_right), and the reverse of the reconstruction,
//      whose four contributions (to the stencil cells k-1 .. k+2) go to LDS;
//   2. each cell adds the contributions of its four faces along the axis
//      and, next to a non-periodic boundary, those that the faces gave the
//      ghost positions copying it (the transpose of the ghost rule; inflow
//      ghosts hold a fixed state and pass nothing on).
// mu = (dR/dU)^T w then enters the stage's adjoint recurrence in the same
// kernel, so no face array or mu array goes through HBM. On a periodic axis
// the faces beyond the grid's ends are evaluated on wrapped stencils: such a
// face is the face on the other side, and the four faces around every cell
// carry all of its contributions.
//
// In 2D the state and the adjoint of the tile and the cells around it are
// staged in LDS once for both axes, and a workgroup of four waves has a thread
// for every face of an axis (19 x 12 and 16 x 15), so each axis is one pass and
// three workgroups fit a CU (54 KB of LDS, 160 registers). The kernel is bound
// by latency, the vector ALU a quarter to half busy. Measured at 512^2 and
// 1024^2, adjoint step: 105 and 281 us; 16 x 13 tiles (two workgroups) 105 and
// 307, 16 x 16 with five waves (one workgroup fits) 124 and 393, 32 x 20 with
// twelve waves 106 and 323; the kernel this replaces (32 x 8 tiles on 256
// threads, whose second pass of each axis had 24 and 96 faces, stencils read
// from global memory, the limiter's cases as branches) 164 and 570.
#include "fv_internal.h"

namespace fvk {

constexpr int ADJ_T = 256;  // threads per workgroup of the 3D kernel, one per tile cell

template <int NDIM>
struct AdjTile;
template <>
struct AdjTile<3> {
    static constexpr int X = 16, Y = 4, Z = 4;
};

// Entries of the face block of axis AX: the tile's extent along the other
// axes times its extent plus three along AX.
template <int NDIM, int AX>
constexpr int adj_faces() {
    using T = AdjTile<NDIM>;
    return (T::X + (AX == 0 ? 3 : 0)) * (T::Y + (AX == 1 ? 3 : 0)) * (T::Z + (AX == 2 ? 3 : 0));
}

template <int NDIM>
constexpr int adj_faces_max() {
    constexpr int a = adj_faces<NDIM, 0>(), b = adj_faces<NDIM, 1>(), c = NDIM == 3 ? adj_faces<NDIM, 2>() : 0;
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

// Cell read at position p along an axis of n cells with face kinds lo / hi
// (0 periodic, 1 transmissive, 2 slip wall, 3 inflow): p itself inside the
// grid; a periodic wrap (any p); the end cell; the mirror cell, with flip set
// (the normal momentum changes sign); -1 behind an inflow face.
__device__ __forceinline__ int adj_src(int p, int n, int lo, int hi, bool& flip) {
    flip = false;
    if (p >= 0 && p < n) return p;
    const bool low = p < 0;
    const int kind = low ? lo : hi;
    if (kind == 0) {
        const int r = p % n;
        return r < 0 ? r + n : r;
    }
    if (kind == 3) return -1;
    if (kind == 2) {
        flip = true;
        return low ? -1 - p : 2 * n - 1 - p;
    }
    return low ? 0 : n - 1;
}

// Steps 1 and 2 above for the faces of axis AX; adds the axis's part of mu
// to acc. o: the tile's first cell, (lx, ly, lz): this thread's cell in
// the tile, own: whether that cell is inside the grid.
template <int NDIM, int AX, int LIM>
__device__ __forceinline__ void adj_axis(const double* __restrict__ Us, const double* __restrict__ w, const Geo& g,
                                         const BcState& bcs, const int* o, int lx, int ly, int lz, bool own,
                                         double ka, double kb, double* C, double* acc) {
    constexpr int NV = NDIM + 2;
    using T = AdjTile<NDIM>;
    constexpr int EX = T::X + (AX == 0 ? 3 : 0), EY = T::Y + (AX == 1 ? 3 : 0), EZ = T::Z + (AX == 2 ? 3 : 0);
    constexpr int NF = EX * EY * EZ;
    const int n = g.n[AX];
    const int lo = g.bc[AX][0], hi = g.bc[AX][1];
    const bool periodic = lo == 0;
    const long long st = AX == 0 ? 1 : (AX == 1 ? g.sy : g.sz);
    const long long wst = AX == 0 ? 1 : (AX == 1 ? g.n[0] : (long long)g.n[0] * g.n[1]);
    // the inflow states of this axis's two faces, read with constant indices
    // and picked per stencil cell by a select (a run-time index into the
    // table would move it to scratch memory)
    double q_lo[NV], q_hi[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        q_lo[v] = bcs.q[AX][0][v];
        q_hi[v] = bcs.q[AX][1][v];
    }
    for (int fi = threadIdx.x; fi < NF; fi += ADJ_T) {
        int p[3];
        p[0] = o[0] + fi % EX;
        p[1] = o[1] + (fi / EX) % EY;
        p[2] = o[2] + fi / (EX * EY);
        p[AX] -= 1;  // the face between cells fpos - 1 and fpos along AX
        const int fpos = p[AX];
        bool live = periodic || (fpos >= 0 && fpos <= n);
#pragma unroll
        for (int d = 0; d < NDIM; ++d)
            if (d != AX) live = live && p[d] < g.n[d];
        double gq[4][NV];
        if (live) {
            p[AX] = 0;
            const long long line = g.off0 + p[0] + (long long)p[1] * g.sy + (long long)p[2] * g.sz;
            const long long wline = ((long long)p[2] * g.n[1] + p[1]) * g.n[0] + p[0];
            double q[4][NV];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int pos = fpos - 2 + s;
                bool flip;
                const int src = adj_src(pos, n, lo, hi, flip);
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    if (src < 0) {
                        q[s][v] = pos < 0 ? q_lo[v] : q_hi[v];
                    } else {
                        const double x = Us[v * g.sv + line + src * st];
                        q[s][v] = (flip && v == 1 + AX) ? -x : x;
                    }
                }
            }
            // the face adds F A to its left cell's residual and -F A to its right cell's
            int cl = fpos - 1, cr = fpos;
            bool hl = cl >= 0, hr = cr < n;
            if (periodic) {
                bool f;
                cl = adj_src(cl, n, 0, 0, f);
                cr = adj_src(cr, n, 0, 0, f);
                hl = hr = true;
            }
            double qL[NV], qR[NV], Fb[NV], qLb[NV], qRb[NV];
            FaceVar<LIM> fv[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const double st4[4] = {q[0][v], q[1][v], q[2][v], q[3][v]};
                fv[v].states(st4, ka, kb, qL[v], qR[v]);
                const double wl = hl ? w[v * (long long)g.ncell + wline + cl * wst] : 0.0;
                const double wr = hr ? w[v * (long long)g.ncell + wline + cr * wst] : 0.0;
                Fb[v] = g.area[AX] * (wl - wr);
            }
            roe_flux_vjp<NDIM, AX>(qL, qR, g.gm1, Fb, qLb, qRb);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                double t[4];
                fv[v].reverse(qLb[v], qRb[v], ka, kb, t);
#pragma unroll
                for (int m = 0; m < 4; ++m) gq[m][v] = t[m];
            }
        } else {
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int v = 0; v < NV; ++v) gq[m][v] = 0.0;
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int v = 0; v < NV; ++v) C[(m * NV + v) * NF + fi] = gq[m][v];
    }
    __syncthreads();
    if (own) {
        const int lp[3] = {lx, ly, lz};
        const int xa = o[AX] + lp[AX];
        // entry of the face block at local face position i along AX, at this cell's other coordinates
        auto fidx = [&](int i) {
            int q[3] = {lx, ly, lz};
            q[AX] = i;
            return q[0] + EX * (q[1] + EY * q[2]);
        };
        // face x + 2 - m (local position lp + 3 - m) holds this cell at stencil slot m
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int e = fidx(lp[AX] + 3 - m);
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] += C[(m * NV + v) * NF + e];
        }
        if (!periodic && (xa < 2 || xa >= n - 2)) {
            // ghosts -2, -1, n, n + 1 that copy this cell
#pragma unroll
            for (int gi = 0; gi < 4; ++gi) {
                const int gp = gi < 2 ? gi - 2 : n + gi - 2;
                const int kind = gi < 2 ? lo : hi;
                if (kind == 3) continue;
                const int src = kind == 2 ? (gi < 2 ? -1 - gp : 2 * n - 1 - gp) : (gi < 2 ? 0 : n - 1);
                if (src != xa) continue;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int f = gp + 2 - m;  // face holding the ghost at slot m
                    const int i = f - o[AX] + 1;
                    if (f < 0 || f > n || i < 0 || i >= (AX == 0 ? EX : (AX == 1 ? EY : EZ))) continue;
                    const int e = fidx(i);
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const double c = C[(m * NV + v) * NF + e];
                        acc[v] += (kind == 2 && v == 1 + AX) ? -c : c;
                    }
                }
            }
        }
    }
    __syncthreads();  // the next axis reuses C
}

// Reverse of the SSP-RK3 stage combinations with L = -R/|Omega|, s = dt/|Omega|,
// mu = (dR/dU_stage)^T w:
//   MODE 3 (w = lam):  lamA = 2/3 lam - 2/3 s mu  (dJ/dU2),  lamB = 1/3 lam
//   MODE 2 (w = lamA): R = 1/4 lamA - 1/4 s mu    (dJ/dU1),  lamB += 3/4 lamA
//   MODE 1 (w = R):    lam = lamB + R - s mu      (dJ/dU^n)
// w is read at the neighbours of a cell, so no stage writes its own w.
template <int MODE>
__device__ __forceinline__ void adj_combine(const double* __restrict__ w, double* lam, double* lamA, double* lamB,
                                            double* R, long long i, double s, double mu) {
    if (MODE == 3) {
        const double l = w[i];
        lamA[i] = (2.0 / 3.0) * l - (2.0 / 3.0) * s * mu;
        lamB[i] = (1.0 / 3.0) * l;
    } else if (MODE == 2) {
        const double a = w[i];
        R[i] = 0.25 * a - 0.25 * s * mu;
        lamB[i] += 0.75 * a;
    } else {
        lam[i] = lamB[i] + w[i] - s * mu;
    }
}

template <int NDIM, int LIM>
__device__ __forceinline__ void adj_axes(const double* __restrict__ Us, const double* __restrict__ w, const Geo& g,
                                         const BcState& bcs, const int* o, int lx, int ly, int lz, bool own,
                                         double ka, double kb, double* C, double* acc) {
    adj_axis<NDIM, 0, LIM>(Us, w, g, bcs, o, lx, ly, lz, own, ka, kb, C, acc);
    adj_axis<NDIM, 1, LIM>(Us, w, g, bcs, o, lx, ly, lz, own, ka, kb, C, acc);
    if constexpr (NDIM == 3) adj_axis<NDIM, 2, LIM>(Us, w, g, bcs, o, lx, ly, lz, own, ka, kb, C, acc);
}

template <int NDIM, int MODE>
__global__ void __launch_bounds__(ADJ_T) k_adj_stage(const double* __restrict__ Us, const double* __restrict__ w,
                                                     double* lam, double* lamA, double* lamB, double* R,
                                                     const double* __restrict__ dtp, Geo g, BcState bcs) {
    constexpr int NV = NDIM + 2;
    using T = AdjTile<NDIM>;
    __shared__ double C[4 * NV * adj_faces_max<NDIM>()];
    const int tiles_x = (g.n[0] + T::X - 1) / T::X, tiles_y = (g.n[1] + T::Y - 1) / T::Y;
    const int b = blockIdx.x;
    const int o[3] = {(b % tiles_x) * T::X, ((b / tiles_x) % tiles_y) * T::Y, (b / (tiles_x * tiles_y)) * T::Z};
    const int t = threadIdx.x;
    const int lx = t % T::X, ly = (t / T::X) % T::Y, lz = t / (T::X * T::Y);
    const int cx = o[0] + lx, cy = o[1] + ly, cz = o[2] + lz;
    const bool own = cx < g.n[0] && cy < g.n[1] && cz < g.n[2];
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    if (g.scheme == 0) {
        adj_axes<NDIM, 0>(Us, w, g, bcs, o, lx, ly, lz, own, 0.0, 0.0, C, acc);
    } else if (g.scheme == 5) {
        adj_axes<NDIM, 3>(Us, w, g, bcs, o, lx, ly, lz, own, 0.0, 0.0, C, acc);
    } else if (g.scheme == 1) {
        adj_axes<NDIM, 1>(Us, w, g, bcs, o, lx, ly, lz, own, 0.0, 0.0, C, acc);
    } else {
        double ka, kb;
        kappa_weights(g.scheme, ka, kb);
        adj_axes<NDIM, 2>(Us, w, g, bcs, o, lx, ly, lz, own, ka, kb, C, acc);
    }
    if (!own) return;
    const double s = *dtp * g.inv_vol;
    const long long e = ((long long)cz * g.n[1] + cy) * g.n[0] + cx;
#pragma unroll
    for (int v = 0; v < NV; ++v)
        adj_combine<MODE>(w, lam, lamA, lamB, R, v * (long long)g.ncell + e, s, acc[v]);
}

// ---------------------------------------------------------------------------
// 2D.

constexpr int A2X = 16, A2Y = 12;            // cells of a tile
constexpr int A2H = 3;                       // cells around it
constexpr int A2RX = A2X + 2 * A2H, A2RY = A2Y + 2 * A2H, A2R = A2RX * A2RY;
constexpr int A2WX = A2X + 4;
constexpr int A2FX = (A2X + 3) * A2Y, A2FY = A2X * (A2Y + 3);  // faces of a pass
constexpr int A2F = A2FX > A2FY ? A2FX : A2FY;
constexpr int A2T = 256;                     // threads: one per face
static_assert(A2F <= A2T && A2X * A2Y <= A2T, "one face per thread and pass");

struct Adj2Lds {
    double U[4][A2R];                        // state of the tile and three cells around it
    double w[4][A2WX * (A2Y + 4)];           // stage adjoint of the tile and two cells around it
    double C[16][A2F];                       // contributions [stencil slot * 4 + variable][face]
};

// One axis: the reverse of this thread's face, then the gather for its cell.
template <int AX, int LIM>
__device__ __forceinline__ void adj2_axis(Adj2Lds& L, const Geo& g, const int* o, double ka, double kb, double* acc) {
    constexpr int EX = AX == 0 ? A2X + 3 : A2X;
    constexpr int st = AX == 0 ? 1 : A2RX;   // neighbour along the axis in the region
    const int t = threadIdx.x;
    const int n = g.n[AX], lo = g.bc[AX][0], hi = g.bc[AX][1];
    const bool periodic = lo == 0;
    {
        // threads past the last face repeat it
        constexpr int NF = AX == 0 ? A2FX : A2FY;
        const int fi = t < NF ? t : NF - 1;
        const int fx = fi % EX, fy = fi / EX;
        // the face between the cells (fx - 2, fx - 1) of the tile on x, or rows (fy - 2, fy - 1)
        const int e = (fy + A2H - (AX == 1 ? 1 : 0)) * A2RX + fx + A2H - (AX == 0 ? 1 : 0);  // its high cell
        constexpr int wst = AX == 0 ? 1 : A2WX;
        const int we = (fy + 2 - (AX == 1 ? 1 : 0)) * A2WX + fx + 2 - (AX == 0 ? 1 : 0);
        const int fpos = o[AX] - 1 + (AX == 0 ? fx : fy);
        const bool live = periodic || (fpos >= 0 && fpos <= n);
        double qL[4], qR[4], Fb[4], qLb[4], qRb[4];
        FaceVar<LIM> fv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double q[4] = {L.U[v][e - 2 * st], L.U[v][e - st], L.U[v][e], L.U[v][e + st]};
            fv[v].states(q, ka, kb, qL[v], qR[v]);
            // the face adds F A to its low cell's residual and -F A to its high cell's
            Fb[v] = g.area[AX] * (L.w[v][we - wst] - L.w[v][we]);
        }
        roe_flux_vjp<2, AX>(qL, qR, g.gm1, Fb, qLb, qRb);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double gq[4];
            fv[v].reverse(qLb[v], qRb[v], ka, kb, gq);
#pragma unroll
            for (int m = 0; m < 4; ++m) L.C[m * 4 + v][fi] = live ? gq[m] : 0.0;
        }
    }
    __syncthreads();
    if (t < A2X * A2Y) {
        const int lx = t % A2X, ly = t / A2X;
        const int xa = o[AX] + (AX == 0 ? lx : ly);
        auto fidx = [&](int i) { return AX == 0 ? ly * EX + i : i * EX + lx; };
        const int lp = AX == 0 ? lx : ly;
        // face x + 2 - m (local position lp + 3 - m) holds this cell at stencil slot m
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int e = fidx(lp + 3 - m);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] += L.C[m * 4 + v][e];
        }
        if (!periodic && (xa < 2 || xa >= n - 2) && xa < n) {
            // ghosts -2, -1, n, n + 1 that copy this cell
#pragma unroll
            for (int gi = 0; gi < 4; ++gi) {
                const int gp = gi < 2 ? gi - 2 : n + gi - 2;
                const int kind = gi < 2 ? lo : hi;
                if (kind == 3) continue;
                const int src = kind == 2 ? (gi < 2 ? -1 - gp : 2 * n - 1 - gp) : (gi < 2 ? 0 : n - 1);
                if (src != xa) continue;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int f = gp + 2 - m;  // face holding the ghost at slot m
                    const int i = f - o[AX] + 1;
                    if (f < 0 || f > n || i < 0 || i >= (AX == 0 ? A2X : A2Y) + 3) continue;
                    const int e = fidx(i);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const double c = L.C[m * 4 + v][e];
                        acc[v] += (kind == 2 && v == 1 + AX) ? -c : c;
                    }
                }
            }
        }
    }
    __syncthreads();  // the next axis reuses C
}

template <int LIM>
__device__ __forceinline__ void adj2_axes(Adj2Lds& L, const Geo& g, const int* o, double ka, double kb, double* acc) {
    adj2_axis<0, LIM>(L, g, o, ka, kb, acc);
    adj2_axis<1, LIM>(L, g, o, ka, kb, acc);
}

// Cell read at position p (adj_src), clamped into the grid further out: any
// number of cells past the ghost layers, which feed no result.
__device__ __forceinline__ int adj2_src(int p, int n, int lo, int hi, bool& flip, int& fixed) {
    flip = false;
    fixed = 0;
    if (p >= 0 && p < n) return p;
    if (lo == 0) {
        while (p < 0) p += n;
        while (p >= n) p -= n;
        return p;
    }
    const int kind = p < 0 ? lo : hi;
    if (kind == 3) fixed = p < 0 ? 1 : 2;
    if (kind == 2 && p >= -2 && p <= n + 1) {
        flip = true;
        return p < 0 ? -1 - p : 2 * n - 1 - p;
    }
    return p < 0 ? 0 : n - 1;
}

template <int MODE>
__global__ void __launch_bounds__(A2T) k_adj_stage2d(const double* __restrict__ Us, const double* __restrict__ w,
                                                     double* lam, double* lamA, double* lamB, double* R,
                                                     const double* __restrict__ dtp, Geo g, BcState bcs) {
    __shared__ Adj2Lds L;
    const int tiles_x = (g.n[0] + A2X - 1) / A2X;
    const int t = threadIdx.x;
    const int o[2] = {(int)(blockIdx.x % tiles_x) * A2X, (int)(blockIdx.x / tiles_x) * A2Y};
    constexpr int IT = (A2R + A2T - 1) / A2T;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int c = t + k * A2T < A2R ? t + k * A2T : A2R - 1;
        const int px = o[0] - A2H + c % A2RX, py = o[1] - A2H + c / A2RX;
        bool fx, fy;
        int qx, qy;
        const int x = adj2_src(px, g.n[0], g.bc[0][0], g.bc[0][1], fx, qx);
        const int y = adj2_src(py, g.n[1], g.bc[1][0], g.bc[1][1], fy, qy);
        const long long p = g.off0 + (long long)y * g.sy + x, e = (long long)y * g.n[0] + x;
        // the stage adjoint is zero outside a non-periodic axis
        const bool out = (g.bc[0][0] != 0 && (px < 0 || px >= g.n[0])) || (g.bc[1][0] != 0 && (py < 0 || py >= g.n[1]));
        const int hx = c % A2RX - 1, hy = c / A2RX - 1, ci = hy * A2WX + hx;
        const bool inner = hx >= 0 && hx < A2WX && hy >= 0 && hy < A2Y + 4;
        double q[4], wv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            q[v] = Us[v * g.sv + p];
            wv[v] = w[v * (long long)g.ncell + e];
        }
        q[1] = fx ? -q[1] : q[1];
        q[2] = fy ? -q[2] : q[2];
        // the inflow states, read with constant indices and picked by selects
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            q[v] = qy == 0 ? q[v] : (qy == 1 ? bcs.q[1][0][v] : bcs.q[1][1][v]);
            q[v] = qx == 0 ? q[v] : (qx == 1 ? bcs.q[0][0][v] : bcs.q[0][1][v]);
            L.U[v][c] = q[v];
            if (inner) L.w[v][ci] = out ? 0.0 : wv[v];
        }
    }
    __syncthreads();
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (g.scheme == 0) {
        adj2_axes<0>(L, g, o, 0.0, 0.0, acc);
    } else if (g.scheme == 5) {
        adj2_axes<3>(L, g, o, 0.0, 0.0, acc);
    } else if (g.scheme == 1) {
        adj2_axes<1>(L, g, o, 0.0, 0.0, acc);
    } else {
        double ka, kb;
        kappa_weights(g.scheme, ka, kb);
        adj2_axes<2>(L, g, o, ka, kb, acc);
    }
    const int cx = o[0] + t % A2X, cy = o[1] + t / A2X;
    if (t >= A2X * A2Y || cx >= g.n[0] || cy >= g.n[1]) return;
    const double s = *dtp * g.inv_vol;
    const long long e = (long long)cy * g.n[0] + cx;
#pragma unroll
    for (int v = 0; v < 4; ++v) adj_combine<MODE>(w, lam, lamA, lamB, R, v * (long long)g.ncell + e, s, acc[v]);
}

// ---------------------------------------------------------------------------

template <int MODE>
static void launch_adj_stage_t(const double* Us, const double* w, double* lam, double* lamA, double* lamB, double* R,
                               const double* dt, const Geo& g, const BcState& bcs, hipStream_t s) {
    if (g.ndim == 2) {
        const long long tiles = (long long)((g.n[0] + A2X - 1) / A2X) * ((g.n[1] + A2Y - 1) / A2Y);
        hipLaunchKernelGGL(k_adj_stage2d<MODE>, dim3((unsigned)tiles), dim3(A2T), 0, s, Us, w, lam, lamA, lamB, R, dt,
                           g, bcs);
        return;
    }
    using T = AdjTile<3>;
    const long long tiles = (long long)((g.n[0] + T::X - 1) / T::X) * ((g.n[1] + T::Y - 1) / T::Y) *
                            ((g.n[2] + T::Z - 1) / T::Z);
    hipLaunchKernelGGL((k_adj_stage<3, MODE>), dim3((unsigned)tiles), dim3(ADJ_T), 0, s, Us, w, lam, lamA, lamB, R, dt,
                       g, bcs);
}

void launch_adj_stage(int mode, const double* Us, const double* w, double* lam, double* lamA, double* lamB, double* R,
                      const double* dt, const Geo& g, const BcState& bcs, hipStream_t s) {
    if (mode == 3) launch_adj_stage_t<3>(Us, w, lam, lamA, lamB, R, dt, g, bcs, s);
    else if (mode == 2) launch_adj_stage_t<2>(Us, w, lam, lamA, lamB, R, dt, g, bcs, s);
    else launch_adj_stage_t<1>(Us, w, lam, lamA, lamB, R, dt, g, bcs, s);
}

}  // namespace fvk
