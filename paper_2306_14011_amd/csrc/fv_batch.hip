// C ABI of the batched fused step: many uneven 2D grids advanced together by
// three fused stage launches per step, captured once in a HIP graph (a
// one-step graph and a graph of GRAPH_STEPS steps, so that a long run pays one
// graph launch per GRAPH_STEPS steps). A batch of several rounds of resident
// waves of large grids is advanced in groups of grids instead (apply_schedule).
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <numeric>
#include <vector>

#include "../../include/fv.h"
#include "fv_internal.h"

namespace {

// Clock record of one step: n entries (even: earliest start, odd: latest
// end), each over fvk::CLK_SLOTS slots.
__global__ void k_clk_reset(unsigned long long* clk, int n) {
    for (int i = threadIdx.x; i < n * fvk::CLK_SLOTS; i += blockDim.x)
        clk[fvk::clk_index(i / fvk::CLK_SLOTS, i % fvk::CLK_SLOTS)] = ((i / fvk::CLK_SLOTS) & 1) ? 0ull : ~0ull;
}

// Folds the slots of this step's clock record into history[counter] and
// advances the counter.
__global__ void k_clk_store(const unsigned long long* clk, int n, unsigned long long* history, int max_steps,
                            int* counter) {
    const int step = *counter;
    if (step < max_steps)
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            unsigned long long v = clk[fvk::clk_index(i, 0)];
            for (int k = 1; k < fvk::CLK_SLOTS; ++k) {
                const unsigned long long w = clk[fvk::clk_index(i, k)];
                v = (i & 1) ? (w > v ? w : v) : (w < v ? w : v);
            }
            history[(long long)step * n + i] = v;
        }
    __syncthreads();
    if (threadIdx.x == 0) *counter = step + 1;
}

__global__ void k_copy_dt(const double* src, double* dst, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

size_t a256(size_t v) { return (v + 255) & ~(size_t)255; }

struct BLayout {
    std::vector<int64_t> offsets;
    int slots;  // wave-speed slots of a grid
    size_t off_fgrid, off_lam, off_dt, off_status, off_clk, off_counter, off_U1, off_U2, total;
};

int validate_batch(int32_t ngrids, const fv_grid_desc* grids, BLayout* L, char* why) {
    if (ngrids < 1 || ngrids > 65536 || !grids) {
        snprintf(why, 256, "ngrids must be in [1, 65536] with a grid array");
        return FV_EINVAL;
    }
    L->offsets.assign(ngrids + 1, 0);
    for (int g = 0; g < ngrids; ++g) {
        const fv_grid_desc& d = grids[g];
        if (d.ndim != 2 || d.n[2] != 1) {
            snprintf(why, 256, "grid %d: batches hold 2D grids only", g);
            return FV_ENOTSUP;
        }
        if (d.n[0] < 1 || d.n[1] < 1 || d.n[0] > 65534 || d.n[1] > 65534) {
            snprintf(why, 256, "grid %d: cell counts must be in [1, 65534]", g);
            return FV_EINVAL;
        }
        if ((int64_t)d.n[0] * d.n[1] * 4 * 8 >= ((int64_t)1 << 32)) {
            snprintf(why, 256, "grid %d: a state of 4 GiB or more (buffer offsets are 32-bit)", g);
            return FV_EINVAL;
        }
        if (d.scheme < FV_SCHEME_MINMOD || d.scheme > FV_SCHEME_QUICK) {
            snprintf(why, 256, "grid %d: unknown scheme", g);
            return FV_EINVAL;
        }
        for (int a = 0; a < 2; ++a) {
            if (!(d.hi[a] > d.lo[a])) {
                snprintf(why, 256, "grid %d: hi must exceed lo", g);
                return FV_EINVAL;
            }
            for (int s = 0; s < 2; ++s) {
                const int kind = d.bc[a][s];
                if (kind != FV_BC_PERIODIC && kind != FV_BC_TRANSMISSIVE && kind != FV_BC_WALL &&
                    kind != FV_BC_INFLOW) {
                    snprintf(why, 256, "grid %d: unknown boundary kind", g);
                    return FV_EINVAL;
                }
                if (kind == FV_BC_WALL && d.n[a] < 2) {
                    snprintf(why, 256, "grid %d: a slip wall needs at least 2 cells on its axis", g);
                    return FV_EINVAL;
                }
                if (kind == FV_BC_INFLOW) {
                    const double* q = d.bc_state[a][s];
                    const double p = (d.gamma - 1.0) * (q[3] - 0.5 * (q[1] * q[1] + q[2] * q[2]) / q[0]);
                    if (!(q[0] > 0.0) || !(p > 0.0) || !isfinite(p)) {
                        snprintf(why, 256, "grid %d: an inflow state needs a positive density and pressure", g);
                        return FV_EINVAL;
                    }
                }
            }
            if ((d.bc[a][0] == FV_BC_PERIODIC) != (d.bc[a][1] == FV_BC_PERIODIC)) {
                snprintf(why, 256, "grid %d: periodic must be set on both faces", g);
                return FV_EINVAL;
            }
        }
        if (!(d.gamma > 1.0) || !(d.cfl > 0.0)) {
            snprintf(why, 256, "grid %d: gamma must exceed 1 and cfl be positive", g);
            return FV_EINVAL;
        }
        if (!(d.mu >= 0.0) || !isfinite(d.mu) || (d.mu > 0.0 && (!(d.prandtl > 0.0) || !isfinite(d.prandtl)))) {
            snprintf(why, 256, "grid %d: viscosity must be finite and >= 0, with a positive Prandtl number", g);
            return FV_EINVAL;
        }
        if (d.nodes) {
            snprintf(why, 256, "grid %d: batches take uniform grids only (no nodes)", g);
            return FV_EINVAL;
        }
        L->offsets[g + 1] = L->offsets[g] + 4 * d.n[0] * d.n[1];
    }
    const size_t total_el = (size_t)L->offsets[ngrids];
    size_t o = 0;
    L->off_fgrid = o;
    o = a256(o + 2 * sizeof(fvk::FGrid) * ngrids);
    L->off_lam = o;
    L->slots = 1;
    for (int g = 0; g < ngrids; ++g) L->slots = std::max(L->slots, fvk::lam_slots(grids[g].n[0] * grids[g].n[1]));
    o = a256(o + fvk::lam_bytes(ngrids, L->slots));
    L->off_dt = o;
    o = a256(o + 8 * (size_t)ngrids);
    L->off_status = o;
    o = a256(o + 4);
    L->off_clk = o;
    o = a256(o + 6 * sizeof(unsigned long long) * fvk::CLK_SLOTS * fvk::CLK_PAD * (size_t)ngrids);
    L->off_counter = o;
    o = a256(o + 4);
    L->off_U1 = o;
    o = a256(o + 8 * total_el);
    L->off_U2 = o;
    o = a256(o + 8 * total_el);
    L->total = o;
    return FV_OK;
}

}  // namespace

struct fv_batch {
    int ngrids, waves, nitems, order;
    int slots;     // wave-speed slots of a grid
    int auto_seg;  // the library's height
    bool own;      // every grid has it, and no wave count is given
    // Parts of the table: the whole batch, then the groups, if there are more than
    // one, that a call of group_steps steps or more advances one after the other.
    struct Group {
        int first, ngrids, nitems;
    };
    std::vector<Group> groups;
    int group_steps;
    int mode;  // stage-kernel variant: 0 periodic / transmissive, 1 walls or inflow faces, 2 viscous
    hipStream_t stream, cap;
    fvk::FGrid* grids;
    unsigned long long* lam;
    double* dt;
    uint32_t* status;
    unsigned long long* clk;
    int* counter;
    double* U1;
    double* U2;
    std::vector<fvk::FGrid> by_grid;     // table entry of each grid, in the caller's order
    std::vector<fvk::FGrid> host_grids;  // the uploaded table, in work-list order
    hipGraph_t graph, graph_many;  // one step; GRAPH_STEPS steps
    hipGraphExec_t exec, exec_many;
    double* graph_U;
    bool graph_timed;
    unsigned long long* graph_history;  // history buffer baked into the captured graph
    unsigned long long* history;
    int max_steps;
    char err[256];
};

static char g_berr[256] = "";

static int bfail(fv_batch* b, int code, const char* msg) {
    snprintf(b ? b->err : g_berr, 256, "%s", msg);
    return code;
}

constexpr int GRAPH_STEPS = 8;

static void drop_graph(fv_batch* b) {
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->exec_many) (void)hipGraphExecDestroy(b->exec_many);
    if (b->graph_many) (void)hipGraphDestroy(b->graph_many);
    b->exec = nullptr;
    b->graph = nullptr;
    b->exec_many = nullptr;
    b->graph_many = nullptr;
    b->graph_U = nullptr;
    b->graph_history = nullptr;
}

// Enqueues the wave speeds of U's grids of group q into cleared slots.
static void enqueue_init(fv_batch* b, const fv_batch::Group& q, const double* U) {
    fvk::launch_fused_init(b->grids + q.first, q.ngrids, q.nitems, U, b->lam, b->status, b->stream, nullptr,
                           b->slots);
}

// Enqueues the three stages of a step of the grids of group q.
static void enqueue_stages(fv_batch* b, const fv_batch::Group& q, double* U, unsigned long long* clk, hipStream_t s) {
    const fvk::FGrid* grids = b->grids + q.first;
    fvk::launch_fused_stage(0, b->waves, grids, q.ngrids, q.nitems, U, U, b->U1, b->lam, b->dt, nullptr, nullptr,
                            b->status, clk, s, nullptr, b->mode, nullptr, b->slots);
    fvk::launch_fused_stage(1, b->waves, grids, q.ngrids, q.nitems, U, b->U1, b->U2, b->lam, b->dt, nullptr, nullptr,
                            b->status, clk, s, nullptr, b->mode, nullptr, b->slots);
    fvk::launch_fused_stage(2, b->waves, grids, q.ngrids, q.nitems, U, b->U2, U, b->lam, b->dt, nullptr, nullptr,
                            b->status, clk, s, nullptr, b->mode, nullptr, b->slots);
}

// Enqueues one step (three stages, plus the clock record when timing) on s. With
// the record, a batch that every call advances in groups takes its groups one
// after the other within the step.
static void enqueue_step(fv_batch* b, double* U, hipStream_t s) {
    const int nclk = 6 * b->ngrids;
    unsigned long long* clk = b->history ? b->clk : nullptr;
    if (clk) hipLaunchKernelGGL(k_clk_reset, dim3(1), dim3(256), 0, s, b->clk, nclk);
    if (clk && b->groups.size() > 1 && b->group_steps == 1)
        for (size_t q = 1; q < b->groups.size(); ++q) enqueue_stages(b, b->groups[q], U, clk, s);
    else
        enqueue_stages(b, b->groups[0], U, clk, s);
    if (clk) hipLaunchKernelGGL(k_clk_store, dim3(1), dim3(256), 0, s, b->clk, nclk, b->history, b->max_steps, b->counter);
}

static bool valid_seg(int32_t seg) { return seg >= 4 && seg <= 1024 && seg % 4 == 0; }

// Splits the grids evenly into as many groups as 24-row items of all of them fill
// the device's resident waves (cap): the largest grid left goes to the group with
// the least work. Where the rounds are nearly full, a group may exceed one by a
// few items (of 954 random batches of up to 96 grids, 14; by 18 items at most) and
// then keeps the batch's segment height. One more group would avoid that, but is
// no faster: 43 grids in three groups of up to 1.015 rounds 665 us a step, in four
// 675. part[g]: the group of grid g.
// Grids of fewer than 20 items on average (some 150 cells a side) stay together.
// steps: the steps of a call from which on groups pay (apply_schedule).
static int split_groups(const std::vector<fvk::FGrid>& grids, long long cap, std::vector<int>& part, int& steps) {
    const int n = (int)grids.size();
    part.assign(n, 0);
    auto items = [&](int g) { return (long long)fvk::fused_items(grids[g], 24); };
    long long total = 0;
    for (int g = 0; g < n; ++g) total += items(g);
    if (cap <= 0 || total <= cap || total < 20LL * n) return 1;
    steps = total < 48LL * n ? 4 : 1;
    std::vector<int> perm(n);
    std::iota(perm.begin(), perm.end(), 0);
    std::stable_sort(perm.begin(), perm.end(), [&](int a, int c) { return items(a) > items(c); });
    const int k = (int)((total + cap - 1) / cap < n ? (total + cap - 1) / cap : n);
    std::vector<long long> load(k, 0);
    for (int g : perm) {
        const int q = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        part[g] = q;
        load[q] += items(g);
    }
    return k;
}

// Orders the table by work-list order, assigns each grid its segment height and
// first work item, and uploads it; the step's graph is rebuilt on the next step.
//
// With the heights at the library's choice, a second table holds the grids in
// groups of one round of resident waves each (split_groups), each with rows of
// its own and its work items counted from 0. A call advances a group by all its
// steps before the next: the waves of a round march in step, so that the halo
// rows they share are still in L2, and a group's states stay in the last-level
// cache from stage to stage and from step to step. That pays for large grids,
// for middling ones in calls of some steps, and not for small ones, which share
// few halo rows and lose at the ends of more launches. us a step, one launch for
// all and in groups, calls of 16, 4 and 1 steps: 96 grids of 128 to 1024 cells a
// side (30M cells) 1700 / 1740 / 1880 and 1580 / 1630 / 1850; 96 of 256^2
// 383 / 388 / 409 and 372 / 380 / 428; 224 of 192^2 505 / 513 / 550 and
// 495 / 513 / 573; 320 of 160^2 482 / 490 / 528 and 483 / 498 / 560; 512 of 128^2
// 583 / 591 / 615 and 576 / 588 / 662; 2048 of 64^2 642 / 646 / 695 and
// 670 / 662 / 735; 8192 of 32^2 655 / 666 / 705 and 731 / 764 / 853; 65536 of 8^2
// 1036 / 1062 / 1139 and 1356 / 1432 / 1732.
static int apply_schedule(fv_batch* b, int32_t order) {
    const int n = b->ngrids;
    std::vector<int> perm(n);
    std::iota(perm.begin(), perm.end(), 0);
    if (order == FV_ORDER_LARGEST_FIRST)
        std::stable_sort(perm.begin(), perm.end(), [&](int a, int c) {
            return (long long)b->by_grid[a].nx * b->by_grid[a].ny > (long long)b->by_grid[c].nx * b->by_grid[c].ny;
        });
    std::vector<int> part(n, 0);
    int k = 1, cus = 0, steps = 1;
    const int per_simd = b->mode == 2 ? 2 : 3;  // resident waves
    if (b->own) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            cus = 0;
        k = split_groups(b->by_grid, 4LL * cus * per_simd, part, steps);
    }
    std::vector<fvk::FGrid> table;
    std::vector<fv_batch::Group> groups;
    // the whole batch, then the groups
    for (int q = k > 1 ? -1 : 0; q < k; ++q) {
        const bool all = groups.empty();
        const int first = (int)table.size();
        for (int g : perm)
            if (all || part[g] == q) table.push_back(b->by_grid[g]);
        fvk::FGrid* grids = table.data() + first;
        const int count = (int)table.size() - first;
        const int rows = b->own ? fvk::fused_rows(grids, count, grids[0].seg, cus, per_simd) : 0;
        long long work = 0;
        for (int i = 0; i < count; ++i) {
            if (rows) grids[i].seg = rows;
            grids[i].work0 = (int)work;
            work += fvk::fused_items(grids[i], grids[i].seg);
        }
        if (work > 0x7fffffff) return bfail(b, FV_EINVAL, "too many work items");
        groups.push_back({first, count, (int)work});
    }
    b->host_grids.swap(table);
    b->groups.swap(groups);
    b->group_steps = steps;
    b->nitems = b->groups[0].nitems;
    b->order = order;
    hipError_t e = hipMemcpyAsync(b->grids, b->host_grids.data(), sizeof(fvk::FGrid) * b->host_grids.size(), hipMemcpyHostToDevice,
                                  b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return bfail(b, FV_EDEVICE, "grid table upload failed");
    drop_graph(b);
    return FV_OK;
}

extern "C" {

int fv_batch_query(int32_t ngrids, const fv_grid_desc* grids, int64_t* offsets, size_t* workspace_bytes) {
    BLayout L;
    int rc = validate_batch(ngrids, grids, &L, g_berr);
    if (rc != FV_OK) return rc;
    if (offsets)
        for (int g = 0; g <= ngrids; ++g) offsets[g] = L.offsets[g];
    if (workspace_bytes) *workspace_bytes = L.total;
    return FV_OK;
}

int fv_batch_create(int32_t ngrids, const fv_grid_desc* grids, int32_t seg, int32_t waves, int32_t order,
                    void* workspace, size_t workspace_bytes, void* stream, fv_batch** out) {
    if (!out) return bfail(nullptr, FV_EINVAL, "null output pointer");
    *out = nullptr;
    BLayout L;
    int rc = validate_batch(ngrids, grids, &L, g_berr);
    if (rc != FV_OK) return rc;
    if (seg != 0 && !valid_seg(seg))
        return bfail(nullptr, FV_EINVAL, "seg must be 0 (automatic) or a multiple of 4 in [4, 1024]");
    if (waves < 0) return bfail(nullptr, FV_EINVAL, "negative wave count");
    if (order != FV_ORDER_GIVEN && order != FV_ORDER_LARGEST_FIRST) return bfail(nullptr, FV_EINVAL, "unknown order");
    if (!workspace || ((uintptr_t)workspace & 255)) return bfail(nullptr, FV_EWORKSPACE, "workspace missing or misaligned");
    if (workspace_bytes < L.total) return bfail(nullptr, FV_EWORKSPACE, "workspace too small");
    fv_batch* b = new (std::nothrow) fv_batch();
    if (!b) return bfail(nullptr, FV_EDEVICE, "host allocation failed");
    b->ngrids = ngrids;
    b->waves = waves;
    b->stream = (hipStream_t)stream;
    char* base = (char*)workspace;
    b->grids = (fvk::FGrid*)(base + L.off_fgrid);
    b->lam = (unsigned long long*)(base + L.off_lam);
    b->dt = (double*)(base + L.off_dt);
    b->status = (uint32_t*)(base + L.off_status);
    b->clk = (unsigned long long*)(base + L.off_clk);
    b->counter = (int*)(base + L.off_counter);
    b->U1 = (double*)(base + L.off_U1);
    b->U2 = (double*)(base + L.off_U2);
    // table entries by grid; each keeps the element offset of its own slot of the state
    b->by_grid.resize(ngrids);
    b->slots = L.slots;
    for (int g = 0; g < ngrids; ++g) {
        const fv_grid_desc& d = grids[g];
        fvk::FGrid& G = b->by_grid[g];
        memset(&G, 0, sizeof(G));
        G.nx = (int)d.n[0];
        G.ny = (int)d.n[1];
        G.pitch = G.nx;
        G.strips = fvk::fused_strips(G.nx);
        G.scheme = d.scheme;
        G.bcx0 = d.bc[0][0];
        G.bcx1 = d.bc[0][1];
        G.bcy0 = d.bc[1][0];
        G.bcy1 = d.bc[1][1];
        G.gid = g;
        G.base = L.offsets[g];
        G.sv = (long long)G.nx * G.ny;
        const double dx = (d.hi[0] - d.lo[0]) / (double)d.n[0];
        const double dy = (d.hi[1] - d.lo[1]) / (double)d.n[1];
        G.ax = dy;
        G.ay = dx;
        G.inv_vol = 1.0 / (dx * dy);
        G.inv_dx = 1.0 / dx;
        G.inv_dy = 1.0 / dy;
        G.cfl = d.cfl;
        G.gamma = d.gamma;
        G.gm1 = d.gamma - 1.0;
        for (int a = 0; a < 2; ++a)
            for (int sd = 0; sd < 2; ++sd)
                for (int v = 0; v < 4; ++v) G.q[a][sd][v] = d.bc_state[a][sd][v];
        G.mu = d.mu;
        if (d.mu > 0.0) {
            G.kcond = d.mu * d.gamma / ((d.gamma - 1.0) * d.prandtl);
            const double hf = d.gamma / d.prandtl;
            G.nu_fac = hf > 4.0 / 3.0 ? hf : 4.0 / 3.0;
        }
        // the stage kernels' variant: viscous if any grid is, else the
        // boundary variant if any grid has a slip wall or an inflow face
        for (int a = 0; a < 2; ++a)
            for (int sd = 0; sd < 2; ++sd)
                if ((d.bc[a][sd] == FV_BC_WALL || d.bc[a][sd] == FV_BC_INFLOW) && b->mode < 1) b->mode = 1;
        if (d.mu > 0.0) b->mode = 2;
    }
    b->auto_seg = fvk::fused_auto_seg(b->by_grid.data(), ngrids, fvk::fused_slots());
    if (seg == 0) seg = b->auto_seg;
    b->own = seg == b->auto_seg && waves == 0;
    for (int g = 0; g < ngrids; ++g) b->by_grid[g].seg = seg;
    hipError_t e = hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking);
    if (e != hipSuccess) {
        snprintf(g_berr, 256, "batch set-up failed: %s", hipGetErrorString(e));
        delete b;
        return FV_EDEVICE;
    }
    rc = apply_schedule(b, order);
    if (rc != FV_OK) {
        snprintf(g_berr, 256, "%s", b->err);
        (void)hipStreamDestroy(b->cap);
        delete b;
        return rc;
    }
    fvk::launch_set_u32(b->status, 0u, b->stream);
    *out = b;
    return FV_OK;
}

int fv_batch_step(fv_batch* b, double* U, int32_t nsteps) {
    if (!b) return bfail(nullptr, FV_EINVAL, "null batch");
    if (!U || nsteps < 0) return bfail(b, FV_EINVAL, "null state or negative step count");
    if (nsteps == 0) return FV_OK;
    const bool timed = b->history != nullptr;
    if (b->groups.size() > 1 && !timed && nsteps >= b->group_steps) {
        // launches of a full round each: no graph needed to hide them
        fvk::launch_lam_reset(b->lam, b->ngrids, b->slots, b->stream);
        for (size_t q = 1; q < b->groups.size(); ++q) {
            enqueue_init(b, b->groups[q], U);
            for (int32_t s = 0; s < nsteps; ++s) enqueue_stages(b, b->groups[q], U, nullptr, b->stream);
        }
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? FV_OK : bfail(b, FV_EDEVICE, hipGetErrorString(e));
    }
    if (b->graph_U != U || !b->exec || b->graph_timed != timed || b->graph_history != b->history) {
        drop_graph(b);
        hipError_t e = hipStreamBeginCapture(b->cap, hipStreamCaptureModeRelaxed);
        if (e == hipSuccess) {
            enqueue_step(b, U, b->cap);
            e = hipStreamEndCapture(b->cap, &b->graph);
        }
        if (e == hipSuccess) e = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0);
        if (e == hipSuccess) e = hipStreamBeginCapture(b->cap, hipStreamCaptureModeRelaxed);
        if (e == hipSuccess) {
            for (int s = 0; s < GRAPH_STEPS; ++s) enqueue_step(b, U, b->cap);
            e = hipStreamEndCapture(b->cap, &b->graph_many);
        }
        if (e == hipSuccess) e = hipGraphInstantiate(&b->exec_many, b->graph_many, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            drop_graph(b);
            return bfail(b, FV_EDEVICE, "graph capture failed");
        }
        b->graph_U = U;
        b->graph_timed = timed;
        b->graph_history = b->history;
    }
    fvk::launch_lam_reset(b->lam, b->ngrids, b->slots, b->stream);
    enqueue_init(b, b->groups[0], U);
    for (int32_t s = 0; s < nsteps;) {
        const bool many = nsteps - s >= GRAPH_STEPS;
        hipError_t e = hipGraphLaunch(many ? b->exec_many : b->exec, b->stream);
        if (e != hipSuccess) return bfail(b, FV_EDEVICE, "graph launch failed");
        s += many ? GRAPH_STEPS : 1;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return bfail(b, FV_EDEVICE, hipGetErrorString(e));
    return FV_OK;
}

int fv_batch_set_timing(fv_batch* b, uint64_t* history, int32_t max_steps, double* ticks_per_us) {
    if (!b) return bfail(nullptr, FV_EINVAL, "null batch");
    if (history && max_steps < 1) return bfail(b, FV_EINVAL, "max_steps must be positive");
    b->history = (unsigned long long*)history;
    b->max_steps = history ? max_steps : 0;
    fvk::launch_set_u32((uint32_t*)b->counter, 0u, b->stream);
    if (ticks_per_us) {
        int dev = 0, khz = 0;
        (void)hipGetDevice(&dev);
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess) khz = 0;
        *ticks_per_us = khz / 1000.0;
    }
    return FV_OK;
}

int fv_batch_dt(fv_batch* b, double* dt) {
    if (!b || !dt) return bfail(b, FV_EINVAL, "null argument");
    hipLaunchKernelGGL(k_copy_dt, dim3(1), dim3(256), 0, b->stream, b->dt, dt, b->ngrids);
    return hipGetLastError() == hipSuccess ? FV_OK : FV_EDEVICE;
}

int fv_batch_status(fv_batch* b, uint32_t* flags) {
    if (!b) return bfail(nullptr, FV_EINVAL, "null batch");
    uint32_t h = 0;
    hipError_t e = hipMemcpyAsync(&h, b->status, sizeof(h), hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return bfail(b, FV_EDEVICE, "status read failed");
    if (flags) *flags = h;
    return h ? FV_ENONPHYS : FV_OK;
}

int fv_batch_set_schedule(fv_batch* b, const int32_t* segs, int32_t order) {
    if (!b) return bfail(nullptr, FV_EINVAL, "null batch");
    if (order != FV_ORDER_GIVEN && order != FV_ORDER_LARGEST_FIRST) return bfail(b, FV_EINVAL, "unknown order");
    if (segs)
        for (int g = 0; g < b->ngrids; ++g)
            if (!valid_seg(segs[g])) return bfail(b, FV_EINVAL, "seg must be a multiple of 4 in [4, 1024]");
    if (segs) {
        for (int g = 0; g < b->ngrids; ++g) b->by_grid[g].seg = segs[g];
        b->own = b->waves == 0 && std::all_of(segs, segs + b->ngrids, [&](int32_t s) { return s == b->auto_seg; });
    }
    return apply_schedule(b, order);
}

int fv_batch_info(const fv_batch* b, int32_t* segs, int32_t* order, int32_t* nitems) {
    if (!b) return FV_EINVAL;
    if (segs)
        for (int g = 0; g < b->ngrids; ++g) segs[g] = b->by_grid[g].seg;
    if (order) *order = b->order;
    if (nitems) *nitems = b->nitems;
    return FV_OK;
}

const char* fv_batch_last_error(const fv_batch* b) { return b ? b->err : g_berr; }

int fv_batch_destroy(fv_batch* b) {
    if (!b) return FV_EINVAL;
    drop_graph(b);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    delete b;
    return FV_OK;
}

}  // extern "C"
