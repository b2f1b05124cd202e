// FP32 kernels of the launch-parameter autotuner's regression network:
// training (forward, backward and Adam over minibatches, one workgroup per 64
// rows of a minibatch, at most eight),
// loss/gradient, prediction, and the exhaustive sweep of the launch space
// with a top-k selection of the lowest predicted runtimes.
//
// Network IN -> 64 -> 64 -> 64 -> 1 with ReLU hidden layers; parameters are
// one flat array W1[64][IN], b1, W2[64][64], b2, W3[64][64], b3, W4[64], b4.
// IN is 14 (the launch features) or 16 (the launch features followed by two
// problem-size features); every kernel is instantiated for both widths.
#include <float.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <mutex>

#include "../../include/fv.h"
#include "fv_device.h"

namespace mlp {

constexpr int H = FV_MLP_HID;

// Offsets of the flat parameter array of the network with IN inputs.
template <int IN>
struct Lay {
    static constexpr int oW1 = 0;
    static constexpr int oB1 = oW1 + H * IN;
    static constexpr int oW2 = oB1 + H;
    static constexpr int oB2 = oW2 + H * H;
    static constexpr int oW3 = oB2 + H;
    static constexpr int oB3 = oW3 + H * H;
    static constexpr int oW4 = oB3 + H;
    static constexpr int oB4 = oW4 + H;
    static constexpr int NP = oB4 + 1;
};
static_assert(Lay<FV_MLP_IN>::NP == FV_MLP_NPARAM, "parameter count");
static_assert(Lay<FV_MLP_IN_SIZED>::NP == FV_MLP_NPARAM_SIZED, "parameter count");
static_assert(FV_MLP_IN_SIZED == FV_MLP_IN + FV_MLP_MAX_EXTRA, "input widths");
constexpr int NP_MAX = Lay<FV_MLP_IN_SIZED>::NP;
constexpr int MAXN = 65536;

// Bytes of scratch that callers pass for n rows. The kernels keep the network,
// the activations and the moments on the chip; training over several
// workgroups exchanges its sums there.
constexpr size_t scratch_bytes(int n) { return ((size_t)5 * n * H + 2 * (size_t)n + NP_MAX) * sizeof(float) + 256; }

// max(z, 0), 0 for NaN, as the median of z, 0 and infinity: one operation. (A
// comparison, fmaxf, and a median with a bound the compiler can see take two,
// the first to quieten a signalling NaN, which sums of products never are.)
__device__ __forceinline__ float relu(float z) {
    float top = __builtin_inff();
    asm("" : "+s"(top));
    return __builtin_amdgcn_fmed3f(z, 0.f, top);
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// Training and gradient: workgroups of eight waves, two per SIMD.
//
// The work of a minibatch is three small matrix products per layer (forward,
// delta, weight gradient) that depend on each other, so the matrix cores of a
// workgroup's CU bound it: 200 rows are 11 MFLOP, 18 us at 256 FP32 operations
// a clock. Everything stays on the chip: the weights and the activations of 128
// rows in LDS, gradients and Adam moments in the registers of the lane that
// holds their sum, so the update needs no exchange. Measured: 200-row
// minibatches in 33 us on one workgroup (18 on four, see Exchange) against
// 530 us for one thread per element with activations and gradients in global
// memory.
//
// Rows go in chunks of 128 (four tiles of 32). Wave w takes tile w / 2 and
// neurons 32 (w % 2) .. + 31 of every layer: transposed products Z^T = W H^T
// (v_mfma_f32_32x32x2f32), whose result holds row l % 32 in every lane l and,
// in register v, neuron 8 (v / 4) + 4 (l / 32) + (v % 4) of the block: four
// registers are four consecutive neurons of a row, one 16-byte LDS access.
// The K order is permuted alike (k_of), so both operands are 16-byte reads
// too. Rows are HS = 68 floats apart: such reads of 16 rows cover the banks.
// Weight gradients are products over the rows (v_mfma_f32_16x16x4f32); wave w
// owns outputs 16 (w % 4) .. + 15 by inputs 32 (w / 4) .. + 31, and the four
// rows of a step are four apart, which makes their reads conflict-free.
// Rows past the minibatch have zero inputs and a zero output delta.
constexpr int TT = 512;      // threads
constexpr int CROWS = 128;   // rows of a chunk
constexpr int HS = 68;       // floats between rows of 64
constexpr int XS = 20;       // floats between rows of inputs

struct alignas(16) TrainLds {
    float Ha[3][CROWS * HS];  // activations of the layers; the third, then the second hold deltas later
    float X[CROWS * XS];      // inputs, 16 per row (zero past IN)
    float W1[H * XS];         // [out][in]
    float W2[H * HS], W3[H * HS];
    float b1[H], b2[H], b3[H], W4[H];
    float b4;
    float y[CROWS], part[2][CROWS], dout[CROWS];
    float red[TT / 64];
    unsigned verdict, lost;  // the exchange's, from thread 0 to all
};

// Sums of a minibatch that a lane owns: tiles of the weight gradients (result
// layout of the 16x16x4 product: output 4 (l / 16) + v, input l % 16), and the
// partial sums over its rows of the other gradients.
struct Grads {
    v4f w3[2], w2[2], w1;
    float b1, b2, b3, w4, b4, sq;
    __device__ void clear() {
        w3[0] = w3[1] = w2[0] = w2[1] = w1 = v4f{};
        b1 = b2 = b3 = w4 = b4 = sq = 0.f;
    }
};

// K index of step s in lane half h.
__device__ __forceinline__ int k_of(int s, int h) { return 8 * (s >> 2) + 4 * h + (s & 3); }

__device__ __forceinline__ v4f ld4(const float* p) { return *(const v4f*)p; }

// z += (rows of W) x (rows of A) over 8 * NQ values of K: W + 8 q + 4 h and
// A + 8 q + 4 h are the lane's operands.
template <int NQ>
__device__ __forceinline__ void mm_rows(const float* W, const float* A, int h, v16f& z) {
    v4f a = ld4(W + 4 * h), b = ld4(A + 4 * h);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        v4f an = a, bn = b;
        if (q + 1 < NQ) {
            an = ld4(W + 8 * (q + 1) + 4 * h);
            bn = ld4(A + 8 * (q + 1) + 4 * h);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) z = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], z, 0, 0, 0);
        a = an;
        b = bn;
        // one pair of operands ahead: its reads hide behind this pair's products
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The block's biases in the result layout.
__device__ __forceinline__ v16f bias16(const float* b, int h) {
    v16f z;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const v4f t = ld4(b + 8 * q + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; ++j) z[4 * q + j] = t[j];
    }
    return z;
}

__device__ __forceinline__ void store16(float* row, int h, const v16f& z) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *(v4f*)(row + 8 * q + 4 * h) = v4f{z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]};
}

// One chunk of nr rows (S.X and S.y filled, a barrier passed): forward, loss,
// backward; adds to g. inv: 1 / rows of the minibatch.
__device__ __forceinline__ void train_chunk(TrainLds& S, int nr, float inv, Grads& g) {
    const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63, h = l >> 5;
    const int tile = wave >> 1, blk = wave & 1;
    const int row = 32 * tile + (l & 31), n0 = 32 * blk, mo = n0 + (l & 31);
    const bool live = 32 * tile < nr;  // uniform: the tile has rows
    const int rows16 = (nr + 15) & ~15;
    float* H1 = S.Ha[0];
    float* H2 = S.Ha[1];
    float* H3 = S.Ha[2];
    v16f z1 = v16f{}, z2 = v16f{};
    if (live) {
        z1 = bias16(S.b1 + n0, h);
        mm_rows<2>(S.W1 + mo * XS, S.X + row * XS, h, z1);
#pragma unroll
        for (int v = 0; v < 16; ++v) z1[v] = relu(z1[v]);
        store16(H1 + row * HS + n0, h, z1);
    }
    __syncthreads();
    if (live) {
        z2 = bias16(S.b2 + n0, h);
        mm_rows<8>(S.W2 + mo * HS, H1 + row * HS, h, z2);
#pragma unroll
        for (int v = 0; v < 16; ++v) z2[v] = relu(z2[v]);
        store16(H2 + row * HS + n0, h, z2);
    }
    __syncthreads();
    if (live) {
        v16f z3 = bias16(S.b3 + n0, h);
        mm_rows<8>(S.W3 + mo * HS, H2 + row * HS, h, z3);
        const v16f w4 = bias16(S.W4 + n0, h);
        float o = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            z3[v] = relu(z3[v]);
            o = fmaf(w4[v], z3[v], o);
        }
        store16(H3 + row * HS + n0, h, z3);
        o += __shfl_xor(o, 32, 64);
        if (h == 0) S.part[blk][row] = o;
    }
    __syncthreads();
    if (tid < CROWS) {
        const float d = tid < nr ? (S.b4 + (S.part[0][tid] + S.part[1][tid])) - S.y[tid] : 0.f;
        S.dout[tid] = d * inv;
        g.sq = fmaf(d, d, g.sq);
    }
    __syncthreads();
    // weight gradients of layer 3 and of the output layer:
    // D3[r][o] = dout_r W4[o] [H3 > 0]
    const int ob = 16 * (wave & 3) + (l & 15), ib = 32 * (wave >> 2) + (l & 15), k4 = 4 * (l >> 4);
    const float w4o = S.W4[ob];
#pragma unroll 4
    for (int s = 0; s < rows16 / 4; ++s) {
        const int r = 16 * (s >> 2) + (s & 3) + k4;
        const float d = S.dout[r], hv = H3[r * HS + ob];
        const float a = hv > 0.f ? d * w4o : 0.f;
        g.w4 = fmaf(d, hv, g.w4);
        g.b3 += a;
        g.b4 += d;
        g.w3[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, H2[r * HS + ib], g.w3[0], 0, 0, 0);
        g.w3[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, H2[r * HS + ib + 16], g.w3[1], 0, 0, 0);
    }
    // D2[r][i] = dout_r sum_o W4[o] W3[o][i] [H3 > 0], where H2 > 0
    v16f dz = v16f{};
    if (live) {
#pragma unroll 2
        for (int q = 0; q < 8; ++q) {
            const v4f hv = ld4(H3 + row * HS + 8 * q + 4 * h), w4 = ld4(S.W4 + 8 * q + 4 * h);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float a = S.W3[(8 * q + 4 * h + j) * HS + mo];
                dz = __builtin_amdgcn_mfma_f32_32x32x2f32(a, hv[j] > 0.f ? w4[j] : 0.f, dz, 0, 0, 0);
            }
        }
        const float d = S.dout[row];
#pragma unroll
        for (int v = 0; v < 16; ++v) dz[v] = z2[v] > 0.f ? d * dz[v] : 0.f;
    }
    __syncthreads();  // every read of H3 and of H2 is done
    if (live) store16(H3 + row * HS + n0, h, dz);
    __syncthreads();
    const float* D2 = H3;
#pragma unroll 4
    for (int s = 0; s < rows16 / 4; ++s) {
        const int r = 16 * (s >> 2) + (s & 3) + k4;
        const float a = D2[r * HS + ob];
        g.b2 += a;
        g.w2[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, H1[r * HS + ib], g.w2[0], 0, 0, 0);
        g.w2[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, H1[r * HS + ib + 16], g.w2[1], 0, 0, 0);
    }
    float* D1 = H2;
    if (live) {
        dz = v16f{};
#pragma unroll 2
        for (int q = 0; q < 8; ++q) {
            const v4f dv = ld4(D2 + row * HS + 8 * q + 4 * h);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                dz = __builtin_amdgcn_mfma_f32_32x32x2f32(S.W2[(8 * q + 4 * h + j) * HS + mo], dv[j], dz, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) dz[v] = z1[v] > 0.f ? dz[v] : 0.f;
        store16(D1 + row * HS + n0, h, dz);
    }
    __syncthreads();
    if (wave < 4) {
#pragma unroll 4
        for (int s = 0; s < rows16 / 4; ++s) {
            const int r = 16 * (s >> 2) + (s & 3) + k4;
            const float a = D1[r * HS + ob];
            g.b1 += a;
            g.w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a, S.X[r * XS + (l & 15)], g.w1, 0, 0, 0);
        }
    }
    __syncthreads();  // the next chunk overwrites X and the activations
}

// A chunk's inputs, requested before the chunk that runs ahead of it: the
// thread's four inputs of row tid / 4 (and the row's target).
template <int IN>
struct RowFetch {
    float x[4], y;
    __device__ void load(const float* __restrict__ X, const float* __restrict__ Y, const int32_t* rows, int base,
                         int nr) {
        const int r = threadIdx.x >> 2, c = 4 * (threadIdx.x & 3);
        const int src = r < nr ? (rows ? rows[base + r] : base + r) : -1;
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = src >= 0 && c + j < IN ? X[(size_t)src * IN + c + j] : 0.f;
        y = src >= 0 ? Y[src] : 0.f;
    }
    __device__ void store(TrainLds& S) const {
        const int r = threadIdx.x >> 2, c = 4 * (threadIdx.x & 3);
        *(v4f*)(S.X + r * XS + c) = v4f{x[0], x[1], x[2], x[3]};
        if (c == 0) S.y[r] = y;
    }
};

template <int IN>
__device__ void load_net(TrainLds& S, const float* __restrict__ P) {
    using L = Lay<IN>;
    for (int e = threadIdx.x; e < H * 16; e += TT) {
        const int o = e >> 4, i = e & 15;
        S.W1[o * XS + i] = i < IN ? P[L::oW1 + o * IN + i] : 0.f;
    }
    for (int e = threadIdx.x; e < H * H; e += TT) {
        S.W2[(e >> 6) * HS + (e & 63)] = P[L::oW2 + e];
        S.W3[(e >> 6) * HS + (e & 63)] = P[L::oW3 + e];
    }
    if (threadIdx.x < H) {
        S.b1[threadIdx.x] = P[L::oB1 + threadIdx.x];
        S.b2[threadIdx.x] = P[L::oB2 + threadIdx.x];
        S.b3[threadIdx.x] = P[L::oB3 + threadIdx.x];
        S.W4[threadIdx.x] = P[L::oW4 + threadIdx.x];
    }
    if (threadIdx.x == 0) S.b4 = P[L::oB4];
}

// Calls f(slot, LDS address, flat index, gradient sum, whether it is a
// weight) for every parameter this lane owns; slots are compile-time
// constants below OWNED.
constexpr int OWNED = 25;
template <int IN, class F>
__device__ __forceinline__ void each_owned(TrainLds& S, Grads& g, F f) {
    using L = Lay<IN>;
    const int wave = threadIdx.x >> 6;
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));  // addresses formed anew at each call: kept across the minibatches, they were spilled
    const int o0 = 16 * (wave & 3) + 4 * (l >> 4), i0 = 32 * (wave >> 2) + (l & 15);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int o = o0 + v, i = i0 + 16 * j;
            f(4 * j + v, &S.W3[o * HS + i], L::oW3 + o * H + i, g.w3[j][v], true);
            f(8 + 4 * j + v, &S.W2[o * HS + i], L::oW2 + o * H + i, g.w2[j][v], true);
        }
    if (wave < 4) {
        if ((l & 15) < IN) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = o0 + v, i = l & 15;
                f(16 + v, &S.W1[o * XS + i], L::oW1 + o * IN + i, g.w1[v], true);
            }
        }
        // the lanes of an output hold partial sums over their rows
        const auto sum4 = [](float t) {
            t += __shfl_xor(t, 16, 64);
            return t + __shfl_xor(t, 32, 64);
        };
        const float b1 = sum4(g.b1), b2 = sum4(g.b2), b3 = sum4(g.b3), w4 = sum4(g.w4), b4 = sum4(g.b4);
        if (l < 16) {
            const int o = 16 * wave + l;
            f(20, &S.b1[o], L::oB1 + o, b1, false);
            f(21, &S.b2[o], L::oB2 + o, b2, false);
            f(22, &S.b3[o], L::oB3 + o, b3, false);
            f(23, &S.W4[o], L::oW4 + o, w4, true);
            if (o == 0) f(24, &S.b4, L::oB4, b4, false);
        }
    }
}

// Sum over the workgroup, in every thread (a barrier on both sides).
__device__ __forceinline__ float block_sum(TrainLds& S, float t) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
    if ((threadIdx.x & 63) == 0) S.red[threadIdx.x >> 6] = t;
    __syncthreads();
    float r = 0.f;
#pragma unroll
    for (int w = 0; w < TT / 64; ++w) r += S.red[w];
    __syncthreads();
    return r;
}

template <int IN>
__global__ void __launch_bounds__(TT) k_loss_grad(const float* __restrict__ P, const float* __restrict__ X,
                                                  const float* __restrict__ Y, int n, float alpha, float* grad,
                                                  float* loss) {
    __shared__ TrainLds S;
    load_net<IN>(S, P);
    Grads g;
    g.clear();
    const float inv = 1.0f / (float)n;
    RowFetch<IN> next;
    next.load(X, Y, nullptr, 0, n);
    for (int c = 0; c < n; c += CROWS) {
        next.store(S);
        __syncthreads();
        if (c + CROWS < n) next.load(X, Y, nullptr, c + CROWS, n - c - CROWS);
        train_chunk(S, min(CROWS, n - c), inv, g);
    }
    const float lam = alpha * inv;
    float w2 = 0.f;
    each_owned<IN>(S, g, [&](int, const float* p, int at, float gs, bool weight) {
        const float w = weight ? *p : 0.f;
        w2 = fmaf(w, w, w2);
        grad[at] = fmaf(lam, w, gs);
    });
    const float t = block_sum(S, 0.5f * inv * (g.sq + alpha * w2));
    if (threadIdx.x == 0) *loss = t;
}

// A minibatch over several workgroups: each takes a share of its rows, all sum
// the shares' gradients in the order of the ranks and make the same Adam step,
// so that each has the whole network and takes the same decision to stop (the
// sums, and with them every later value, are the same bits in all).
// Bound by the chain forward - backward - exchange - update: 64 rows take 13 us
// on one workgroup, of which some 6 are matrix products, and the exchange of
// 43 KB a workgroup through the last-level cache 4.6 us more, so that a
// workgroup takes up to 64 rows before another is added. 200-row minibatches:
// 33.3 us on one workgroup, 22.1 on two, 17.9 on four; 500 rows 73, 42, 26, and
// 21.2 on eight; 128 rows 20.5, and 16.4 on two. (Fences in every thread in
// place of one cost 2.4 us more, and 64 rows then took 13.0 us on one and 16.8
// on two. All workgroups on one XCD take 1 us less, but would queue the
// trainings of several streams on its 32 CUs.)
// A workgroup waits for others only once all of a launch are known to be
// resident: they may not be (other launches or processes hold CUs, or a graph
// that was captured here is replayed on a stream of fewer CUs), and one that
// waits for another that its own CU would have to run never ends. So a launch
// begins with a roll call: whoever arrives last makes it TOGETHER, and whoever
// has waited long enough makes it STAND_ALONE, in which all leave and a launch
// of one workgroup behind it computes every rank's share, one after another.
// Both give the same bits.
// Resident workgroups stay so, which ends the later waits; they are bounded too
// (a second call on the same scratch breaks them), and a call that loses one
// reports it and leaves the network as it was.
// Rank r goes to XCD r, so that 32 launches are resident whole before one could
// be in part. A stream that may not use every CU of the device, and a device of
// fewer than 64, take one workgroup.
constexpr int MAX_WGS = 8;
constexpr int WG_ROWS = 64;

static int train_workgroups(int batch, hipStream_t stream) {
    const int w = (batch + WG_ROWS - 1) / WG_ROWS;
    if (w < 2) return 1;
    int dev = 0, cus = 0, usable = 0;
    uint32_t mask[32] = {};
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipExtStreamGetCUMask(stream, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    for (uint32_t m : mask) usable += __builtin_popcount(m);
    if (cus < 64 || usable < cus) return 1;
    return w < MAX_WGS ? w : MAX_WGS;
}

// Polls of a counter (0.14 us each) before a wait is given up: some 40 ms for
// the roll call, which no launch that finds the CUs free needs, and 5 s between
// resident workgroups, which take microseconds. They count the time that the
// workgroup runs, so a process that is set aside loses nothing.
constexpr int ROLL_POLLS = 1 << 18;
constexpr int WAIT_POLLS = 1 << 25;

// Exchange buffer, in the caller's scratch (from a multiple of 64 bytes on): four
// words in lines of their own, then per workgroup its sums of a minibatch as
// every lane holds them: four vectors of four, and for the lanes of the first
// four waves two more and two values.
enum { EX_SENT = 0, EX_ARRIVED = 16, EX_TAKEN = 32, EX_VERDICT = 48 };
enum { TOGETHER = 1, STAND_ALONE = 2 };
constexpr size_t EX_HEAD = 256;
constexpr size_t EX_ROW = TT * 16;                                // bytes of a vector of every lane
constexpr size_t EX_BYTES = 4 * EX_ROW + TT / 2 * (16 + 16 + 8);  // 43008 per workgroup
constexpr bool exchange_fits() {
    for (int w = 2; w <= MAX_WGS; ++w)
        if (64 + EX_HEAD + w * EX_BYTES > scratch_bytes(WG_ROWS * (w - 1) + 1)) return false;
    return true;
}
static_assert(exchange_fits(), "the scratch of the smallest batch for a number of workgroups holds their sums");

struct Exchange {
    char* base;
    int rank, size;
    int polls;       // the bound of a wait between resident workgroups
    unsigned sent, taken;  // what the counters reach when all have written, and have read, a minibatch's sums

    __device__ unsigned* word(int at) const { return (unsigned*)base + at; }
    // Whether the counter reached count within the bound.
    __device__ bool wait(int at, unsigned count) const {
        for (int i = 0; i < polls; ++i) {
            if ((int)(__hip_atomic_load(word(at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - count) >= 0) return true;
            __builtin_amdgcn_s_sleep(1);
        }
        return false;
    }
    // Thread 0: says that this workgroup is resident (with bound 0: none is called).
    __device__ void arrive(int bound) const {
        if (bound > 0 && __hip_atomic_fetch_add(word(EX_ARRIVED), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
                             (unsigned)size)
            decide(TOGETHER);
    }
    // The first verdict of the launch stands.
    __device__ unsigned decide(unsigned verdict) const {
        unsigned first = 0;
        return __hip_atomic_compare_exchange_strong(word(EX_VERDICT), &first, verdict, __ATOMIC_RELAXED,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   ? verdict
                   : first;
    }
    // Thread 0: the verdict, which all workgroups see alike.
    __device__ unsigned roll_call(int bound) const {
        for (int i = 0; i < bound; ++i) {
            const unsigned v = __hip_atomic_load(word(EX_VERDICT), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v != 0) return v;
            __builtin_amdgcn_s_sleep(1);
        }
        return decide(STAND_ALONE);
    }
    // Before a barrier after which one thread tells the other workgroups that all
    // waves' sums are written, or read: a wave counts only its own outstanding
    // accesses, and the barrier waits for none, so each waits for its own here.
    // The one thread's write-back and count then come after all of them. (The
    // fence in every thread would do too, with eight write-backs of the L2: see
    // above.)
    __device__ static void settle() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

    // Writes g as the sums of rank r.
    __device__ void put(const Grads& g, int r) const {
        const int tid = threadIdx.x;
        char* const out = base + EX_HEAD + r * EX_BYTES + tid * 16;
        *(v4f*)out = g.w3[0];
        *(v4f*)(out + EX_ROW) = g.w3[1];
        *(v4f*)(out + 2 * EX_ROW) = g.w2[0];
        *(v4f*)(out + 3 * EX_ROW) = g.w2[1];
        if (tid < TT / 2) {  // uniform over a wave
            *(v4f*)(out + 4 * EX_ROW) = g.w1;
            *(v4f*)(out + 4 * EX_ROW + TT / 2 * 16) = v4f{g.b1, g.b2, g.b3, g.w4};
            *(float2*)(base + EX_HEAD + r * EX_BYTES + 4 * EX_ROW + TT * 16 + tid * 8) = float2{g.b4, g.sq};
        }
    }
    // g: the sums of all ranks, in their order (every lane reads what its like wrote).
    __device__ void take(Grads& g) const {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // addresses formed anew at each call, as in each_owned (in put it cost 1.5 us a minibatch)
        g.clear();
#pragma unroll 1
        for (int r = 0; r < size; ++r) {
            const char* const in = base + EX_HEAD + r * EX_BYTES + tid * 16;
            g.w3[0] += *(const v4f*)in;
            g.w3[1] += *(const v4f*)(in + EX_ROW);
            g.w2[0] += *(const v4f*)(in + 2 * EX_ROW);
            g.w2[1] += *(const v4f*)(in + 3 * EX_ROW);
            if (tid < TT / 2) {
                g.w1 += *(const v4f*)(in + 4 * EX_ROW);
                const v4f b = *(const v4f*)(in + 4 * EX_ROW + TT / 2 * 16);
                g.b1 += b[0];
                g.b2 += b[1];
                g.b3 += b[2];
                g.w4 += b[3];
                const float2 c = *(const float2*)(base + EX_HEAD + r * EX_BYTES + 4 * EX_ROW + TT * 16 + tid * 8);
                g.b4 += c.x;
                g.sq += c.y;
            }
        }
    }
    // Sums g over the workgroups, in all of them; false (in every thread): a wait was given up.
    __device__ bool sum(TrainLds& S, Grads& g) {
        const bool first = threadIdx.x == 0;
        // every workgroup has read the previous minibatch's sums
        if (first && !wait(EX_TAKEN, taken)) S.lost = 1;
        __syncthreads();
        put(g, rank);
        settle();
        __syncthreads();
        sent += size;
        taken += size;
        if (first) {
            __hip_atomic_fetch_add(word(EX_SENT), 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            if (!wait(EX_SENT, sent)) S.lost = 1;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        take(g);
        const int lost = __builtin_amdgcn_readfirstlane((int)S.lost);
        settle();
        __syncthreads();
        if (first) __hip_atomic_fetch_add(word(EX_TAKEN), 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        return lost == 0;
    }
};

// Clears the counters (a kernel, so that the call can be captured in a graph).
__global__ void k_train_clear(unsigned* ctr) { ctr[threadIdx.x] = 0; }

// ALONE: the launch of one workgroup that follows a shared one and computes
// the shares of all its `size` ranks, one after another, where the roll call
// says so; else it ends at once. (In one kernel with the shared path, which
// fills the registers, that path took 0.4 to 1.5 us more a minibatch; the second
// launch takes 2 us of a call.)
template <int IN, bool ALONE>
__global__ void __launch_bounds__(TT) k_train(float* P, float* M, float* V, int32_t* tptr, const float* __restrict__ X,
                                              const float* __restrict__ Y, int n, const int32_t* __restrict__ order,
                                              fv_mlp_hparams hp, float* epoch_loss, int32_t* epochs_run, char* exchange,
                                              int size, int roll_polls, int wait_polls) {
    __shared__ TrainLds S;
    const int rank = ALONE ? 0 : blockIdx.x;
    Exchange ex{exchange, rank, size, wait_polls, 0, 0};
    if (ALONE && *ex.word(EX_VERDICT) != STAND_ALONE) return;
    if (hp.max_epochs <= 0) {
        if (rank == 0 && threadIdx.x == 0) *epochs_run = 0;
        return;
    }
    if (!ALONE && size > 1 && threadIdx.x == 0) ex.arrive(roll_polls);
    int t = *tptr;
    // running powers of the decay factors for the bias correction
    double p1 = pow((double)hp.beta1, (double)t), p2 = pow((double)hp.beta2, (double)t);
    load_net<IN>(S, P);
    Grads g;
    g.clear();
    float m[OWNED], v[OWNED];
    each_owned<IN>(S, g, [&](int k, const float*, int at, float, bool) {
        m[k] = M[at];
        v[k] = V[at];
    });
    if (!ALONE && size > 1) {
        if (threadIdx.x == 0) {
            S.verdict = ex.roll_call(roll_polls);
            S.lost = 0;
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane((int)S.verdict) != TOGETHER) return;
    }
    float best = FLT_MAX;
    int noimp = 0;
    int e = 0;
    // Rank r's rows of a minibatch of sz rows: part of them, from lo.
    auto lo = [&](int sz, int r) { return (int)((long long)sz * r / size); };
    auto part = [&](int sz, int r) { return (int)((long long)sz * (r + 1) / size) - lo(sz, r); };
    RowFetch<IN> next;
    {
        const int sz = min(hp.batch, n);
        next.load(X, Y, order, lo(sz, rank), part(sz, rank));
    }
    for (; e < hp.max_epochs; ++e) {
        float acc = 0.f;  // this lane's part of the epoch's loss
        const int32_t* rows = order + (size_t)e * n;
        for (int start = 0; start < n; start += hp.batch) {
            const int sz = min(hp.batch, n - start);
            const float inv = 1.0f / (float)sz;
            int r = rank;
            do {
                const int own = part(sz, r);
                g.clear();
                for (int c = 0; c == 0 || c < own; c += CROWS) {
                    next.store(S);
                    __syncthreads();
                    // the following chunk: of this share, of the next one, of the next minibatch, or of the next epoch
                    if (c + CROWS < own) {
                        next.load(X, Y, rows, start + lo(sz, r) + c + CROWS, own - c - CROWS);
                    } else if (ALONE && r + 1 < size) {
                        next.load(X, Y, rows, start + lo(sz, r + 1), part(sz, r + 1));
                    } else if (start + sz < n) {
                        const int nsz = min(hp.batch, n - start - sz);
                        next.load(X, Y, rows, start + sz + lo(nsz, rank), part(nsz, rank));
                    } else if (e + 1 < hp.max_epochs) {
                        const int nsz = min(hp.batch, n);
                        next.load(X, Y, rows + n, lo(nsz, rank), part(nsz, rank));
                    }
                    train_chunk(S, min(CROWS, own - c), inv, g);
                }
                if (ALONE) ex.put(g, r);
            } while (ALONE && ++r < size);
            if (ALONE) {
                ex.take(g);
            } else if (size > 1 && !ex.sum(S, g)) {
                if (rank == 0 && threadIdx.x == 0) *epochs_run = -1;
                return;
            }
            ++t;
            p1 *= (double)hp.beta1;
            p2 *= (double)hp.beta2;
            const float lrt = (float)((double)hp.lr * sqrt(1.0 - p2) / (1.0 - p1));
            const float lam = hp.alpha * inv;
            float w2 = 0.f;
            each_owned<IN>(S, g, [&](int k, float* p, int, float gs, bool weight) {
                const float w = *p, gr = weight ? fmaf(lam, w, gs) : gs;
                if (weight) w2 = fmaf(w, w, w2);
                m[k] = hp.beta1 * m[k] + (1.f - hp.beta1) * gr;
                v[k] = hp.beta2 * v[k] + (1.f - hp.beta2) * gr * gr;
                *p = w - lrt * m[k] / (sqrtf(v[k]) + hp.eps);
                // (all parameters' roots and quotients at once would take more registers than there are)
                if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            });
            acc += 0.5f * (g.sq + hp.alpha * w2);  // the minibatch's loss times its rows
            // (the next chunk's barrier publishes the new weights)
        }
        const float el = block_sum(S, acc) / (float)n;
        if (rank == 0 && threadIdx.x == 0) epoch_loss[e] = el;
        if (el > best - hp.tol) ++noimp;
        else noimp = 0;
        if (el < best) best = el;
        if (noimp > hp.n_iter_no_change) {
            ++e;
            break;
        }
    }
    if (rank != 0) return;
    g.clear();
    each_owned<IN>(S, g, [&](int k, const float* p, int at, float, bool) {
        P[at] = *p;
        M[at] = m[k];
        V[at] = v[k];
    });
    if (threadIdx.x == 0) {
        *epochs_run = e;
        *tptr = t;
    }
}

// ---------------------------------------------------------------------------
// Sweep of the launch space.

constexpr int KMAX = 8;
constexpr int SWEEP_T = 256;
constexpr int SWEEP_MAXB = 4096;

struct SweepTab {
    int32_t radix[FV_NSITES];
    float f[2][FV_NSITES][FV_SPACE_MAXC];  // the two features of a site's choice
    float extra[FV_MLP_MAX_EXTRA];
};

// (v, i) orders before (w, j): lower value, ties to the lower index; NaN last.
__device__ __forceinline__ bool before(float v, long long i, float w, long long j) {
    return v < w || (v == w && i < j);
}

// Thread-local ascending top-k list.
struct TopK {
    float v[KMAX];
    long long i[KMAX];
    __device__ void init() {
#pragma unroll
        for (int q = 0; q < KMAX; ++q) {
            v[q] = FLT_MAX;
            i[q] = LLONG_MAX;
        }
    }
    __device__ void insert(float val, long long idx) {
        if (!(val == val)) val = FLT_MAX;  // NaN never wins
        if (!before(val, idx, v[KMAX - 1], i[KMAX - 1])) return;
        float cv = val;
        long long ci = idx;
#pragma unroll
        for (int q = 0; q < KMAX; ++q) {
            if (before(cv, ci, v[q], i[q])) {
                const float tv = v[q];
                const long long ti = i[q];
                v[q] = cv;
                i[q] = ci;
                cv = tv;
                ci = ti;
            }
        }
    }
};

// The k best of the workgroup's lists in ascending order, in out(round, value,
// index) calls of thread 0: the lists are sorted, so each round compares their
// heads and the winner's list moves up. NW: waves. (Rounds over all entries in
// memory took 70 us for the lists of 4096 workgroups, 10 % of a sweep of 2M.)
template <int NW>
struct TopkLds {
    float v[2][NW];
    long long i[2][NW];
};

template <int NW, class F>
__device__ __forceinline__ void block_topk(TopK& top, int k, TopkLds<NW>& S, F out) {
    const int w = threadIdx.x >> 6;
    for (int round = 0; round < k; ++round) {
        float bv = top.v[0];
        long long bi = top.i[0];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(bv, off, 64);
            const long long oi = __shfl_xor(bi, off, 64);
            if (before(ov, oi, bv, bi)) {
                bv = ov;
                bi = oi;
            }
        }
        const int s = round & 1;  // two sets: one barrier a round
        if ((threadIdx.x & 63) == 0) {
            S.v[s][w] = bv;
            S.i[s][w] = bi;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NW; ++q)
            if (before(S.v[s][q], S.i[s][q], bv, bi)) {
                bv = S.v[s][q];
                bi = S.i[s][q];
            }
        if (threadIdx.x == 0) out(round, bv, bi);
        if (top.i[0] == bi) {  // indices are unique (but for the end marks, which follow one another)
#pragma unroll
            for (int q = 0; q + 1 < KMAX; ++q) {
                top.v[q] = top.v[q + 1];
                top.i[q] = top.i[q + 1];
            }
            top.v[KMAX - 1] = FLT_MAX;
            top.i[KMAX - 1] = LLONG_MAX;
        }
    }
}

// The sweep on the matrix cores. A wave takes 32 configurations at a time and
// runs the network in transposed form, Z^T = W H^T, with
// v_mfma_f32_32x32x2f32: M = 32 neurons of a block (two blocks per 64-wide
// layer), N = the 32 configurations, K = 2 inputs per instruction. Operand
// lanes: A (32 x 2) has neuron l % 32 and input l / 32, B (2 x 32) input
// l / 32 and configuration l % 32; the 32 x 32 result holds configuration
// l % 32 in every lane and, in register v, neuron 8 (v / 4) + 4 (l / 32) +
// (v % 4). So the activations never move: the next layer takes register v of
// block b as one K pair (lanes 0-31 and 32-63 hold different neurons), and its
// weight operand is permuted to the same neuron order. Each layer's bias is
// one more K step with inputs (1, 0). The weight operands are staged once per
// workgroup in LDS, in the instruction's lane order; the sums run in another
// order than the row-per-thread forward pass (FP32 rounding apart, the same
// network). Bound by the matrix cores (148 instructions of 64 cycles a tile,
// 90 % of the time; what is left is the 215 vector operations between them):
// 189M configurations of 14 inputs in 25.9 ms, 134 TFLOP/s; 28.8 with the
// choices by division (4 %), results in accumulation registers that vector
// operations cannot read and two operations per ReLU (4 %), and the longer
// staging and selection (2 %).
template <int IN>
struct MfLds {
    static constexpr int S1 = IN / 2;                  // K steps of layer 1 (IN is even)
    static constexpr int A1 = 0;                       // [block][step 0 .. S1][lane]
    static constexpr int A2 = A1 + 2 * (S1 + 1) * 64;  // [block][step 0 .. 32][lane]
    static constexpr int A3 = A2 + 2 * 33 * 64;
    static constexpr int W4 = A3 + 2 * 33 * 64;        // [block * 16 + register][lane]
    static constexpr int FLOATS = W4 + 32 * 64;
};

// Neuron of register v of block b in lane half h of a result.
__device__ __forceinline__ int mf_neuron(int b, int v, int h) { return 32 * b + 8 * (v >> 2) + 4 * h + (v & 3); }

// One layer: c[b] = sum over the NST K steps of A (block b, step st) times
// bval(st), the two blocks interleaved. The steps go in groups of four whose
// weight operands are read from LDS while the previous group's instructions
// issue; the scheduling barrier keeps the compiler from hoisting every read
// of the layer (and the registers they take) to its start.
template <int NST, int AOFF, class BF>
__device__ __forceinline__ void mf_layer(const float* A, int lane, BF bval, v16f* c) {
    constexpr int G = 4;
    c[0] = v16f{};
    c[1] = v16f{};
    float a[2][2 * G];
#pragma unroll
    for (int q = 0; q < G; ++q)
        if (q < NST)
#pragma unroll
            for (int b = 0; b < 2; ++b) a[0][2 * q + b] = A[AOFF + (b * NST + q) * 64 + lane];
#pragma unroll
    for (int g = 0; g * G < NST; ++g) {
        const int cur = g & 1;
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int st = (g + 1) * G + q;
            if (st < NST)
#pragma unroll
                for (int b = 0; b < 2; ++b) a[cur ^ 1][2 * q + b] = A[AOFF + (b * NST + st) * 64 + lane];
        }
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int st = g * G + q;
            if (st < NST) {
                const float bv = bval(st);
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    c[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][2 * q + b], bv, c[b], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The weight operands of the network in LDS, in the instruction's lane order.
// Read along the rows of the matrices, all of a thread's loads at once, and
// scattered in LDS (each write of a row meets two banks): in the operands'
// order, a wave's load touched 64 lines and the threads' 45 loads followed one
// another, 15 us of a sweep's or prediction's 18.
template <int IN>
__device__ __forceinline__ void stage_net(float* A, const float* __restrict__ P) {
    using L = Lay<IN>;
    using M = MfLds<IN>;
    constexpr int PER = H * H / SWEEP_T;
    const int t = threadIdx.x;
    float w2[PER], w3[PER], w1[H * IN / SWEEP_T + 1];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        w2[q] = P[L::oW2 + t + q * SWEEP_T];
        w3[q] = P[L::oW3 + t + q * SWEEP_T];
    }
#pragma unroll
    for (int q = 0; q * SWEEP_T < H * IN; ++q)
        w1[q] = t + q * SWEEP_T < H * IN ? P[L::oW1 + t + q * SWEEP_T] : 0.f;
    // biases, one K step each: lane half 0 (lane half 1 meets an input of 0)
    const float b1 = P[L::oB1 + t % H], b2 = P[L::oB2 + t % H], b3 = P[L::oB3 + t % H];
    float w4[32 * 64 / SWEEP_T];
#pragma unroll
    for (int q = 0; q < 32 * 64 / SWEEP_T; ++q) {
        const int e = t + q * SWEEP_T, r = e >> 6;
        w4[q] = P[L::oW4 + mf_neuron(r >> 4, r & 15, (e >> 5) & 1)];
    }
    // input neuron i of a layer is the K step 16 (i / 32) + 4 (i % 32 / 8) + i % 4 of lane half i / 4 % 2
    const int i = t % H, st = 16 * (i >> 5) + 4 * ((i & 31) >> 3) + (i & 3), l = 32 * ((i >> 2) & 1);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int m = t / H + q * (SWEEP_T / H);
        const int at = ((m >> 5) * 33 + st) * 64 + l + (m & 31);
        A[M::A2 + at] = w2[q];
        A[M::A3 + at] = w3[q];
    }
#pragma unroll
    for (int q = 0; q * SWEEP_T < H * IN; ++q) {
        const int e = t + q * SWEEP_T, m = e / IN, k = e % IN;
        if (e < H * IN) A[M::A1 + ((m >> 5) * (M::S1 + 1) + (k >> 1)) * 64 + 32 * (k & 1) + (m & 31)] = w1[q];
    }
    if (t < 2 * H) {
        const int m = t % H, half = t / H, at = (m >> 5) * 64 + 32 * half + (m & 31);
        A[M::A1 + (m >> 5) * M::S1 * 64 + M::S1 * 64 + at] = half ? 0.f : b1;
        A[M::A2 + (m >> 5) * 32 * 64 + 32 * 64 + at] = half ? 0.f : b2;
        A[M::A3 + (m >> 5) * 32 * 64 + 32 * 64 + at] = half ? 0.f : b3;
    }
#pragma unroll
    for (int q = 0; q < 32 * 64 / SWEEP_T; ++q) A[M::W4 + t + q * SWEEP_T] = w4[q];
}

// The network's output for the row in lane l % 32, whose inputs are x, in both lane halves.
template <int IN>
__device__ __forceinline__ float mf_forward(const float* A, int lane, const float* x, float b4) {
    using M = MfLds<IN>;
    const int h = lane >> 5;
    const float one = h == 0 ? 1.f : 0.f;
    v16f c1[2], c2[2], c3[2];
    mf_layer<M::S1 + 1, M::A1>(A, lane, [&](int st) { return st < M::S1 ? (h ? x[2 * st + 1] : x[2 * st]) : one; },
                               c1);
    mf_layer<33, M::A2>(A, lane, [&](int st) { return st < 32 ? relu(c1[st >> 4][st & 15]) : one; }, c2);
    mf_layer<33, M::A3>(A, lane, [&](int st) { return st < 32 ? relu(c2[st >> 4][st & 15]) : one; }, c3);
    float part = 0.f;
#pragma unroll
    for (int q = 0; q < 32; ++q) part = fmaf(A[M::W4 + q * 64 + lane], relu(c3[q >> 4][q & 15]), part);
    return b4 + (part + __shfl_xor(part, 32, 64));
}

// Predictions of n rows, 32 to a wave. (One thread per row with the weights as
// scalar operands took 112 us for 500 rows, a chain of scalar loads in 8
// waves; 12 us here, most of it the staging of the weights.)
template <int IN>
__global__ void __launch_bounds__(SWEEP_T) __attribute__((amdgpu_waves_per_eu(3))) k_predict(const float* __restrict__ P, const float* __restrict__ X, int n,
                                                     float* __restrict__ out) {
    __shared__ __align__(16) float A[MfLds<IN>::FLOATS];
    const int lane = threadIdx.x & 63;
    const int r = (blockIdx.x * (SWEEP_T / 64) + (threadIdx.x >> 6)) * 32 + (lane & 31);
    const int src = r < n ? r : n - 1;
    float x[IN];
#pragma unroll
    for (int i = 0; i < IN; ++i) x[i] = X[(size_t)src * IN + i];
    stage_net<IN>(A, P);
    __syncthreads();
    const float o = mf_forward<IN>(A, lane, x, P[Lay<IN>::oB4]);
    if (lane < 32 && r < n) out[r] = o;
}

template <int IN>
__global__ void __launch_bounds__(SWEEP_T) __attribute__((amdgpu_waves_per_eu(3))) k_sweep_mfma(const float* __restrict__ P, SweepTab tab, long long begin,
                                                         long long count, int k, float* __restrict__ pv,
                                                         long long* __restrict__ pi) {
    using L = Lay<IN>;
    using M = MfLds<IN>;
    static_assert(IN % 2 == 0, "layer 1 takes inputs in pairs");
    __shared__ __align__(16) float A[M::FLOATS];
    __shared__ TopkLds<SWEEP_T / 64> S;
    stage_net<IN>(A, P);
    __syncthreads();
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const float one = h == 0 ? 1.f : 0.f;
    const float b4 = P[L::oB4];
    TopK top;
    top.init();
    const long long tiles = (count + 31) / 32;
    const long long nw = (long long)gridDim.x * (SWEEP_T / 64);
    const long long t0 = (long long)blockIdx.x * (SWEEP_T / 64) + (threadIdx.x >> 6);
    // The choices of this lane's configuration, the digits of its index, and
    // those of the distance to the wave's next one: added digit by digit from
    // tile to tile (a 64-bit division per site and tile took 4 % of the
    // sweep). Past the space's end they wrap, and stay choices.
    unsigned digit[FV_NSITES], step[FV_NSITES];
    {
        unsigned long long at = (unsigned long long)(begin + t0 * 32 + (lane & 31)), by = (unsigned long long)nw * 32;
#pragma unroll
        for (int site = 0; site < FV_NSITES; ++site) {
            const unsigned rd = (unsigned)tab.radix[site];
            digit[site] = (unsigned)(at % rd);
            at /= rd;
            step[site] = (unsigned)(by % rd);
            by /= rd;
        }
    }
    for (long long t = t0; t < tiles; t += nw) {
        // layer 1's inputs in pairs: this lane half's of each
        float x[IN / 2];
#pragma unroll
        for (int site = 0; site < FV_NSITES; ++site) x[site] = tab.f[h][site][digit[site]];
#pragma unroll
        for (int j = FV_NSITES; j < IN / 2; ++j) x[j] = tab.extra[2 * (j - FV_NSITES) + h];
        unsigned carry = 0;
#pragma unroll
        for (int site = 0; site < FV_NSITES; ++site) {
            const unsigned rd = (unsigned)tab.radix[site], d = digit[site] + step[site] + carry;
            carry = d >= rd ? 1u : 0u;
            digit[site] = min(d, d - rd);  // d - rd wraps to above d below the radix
        }
        v16f c1[2], c2[2], c3[2];
        mf_layer<M::S1 + 1, M::A1>(A, lane, [&](int st) { return st < M::S1 ? x[st] : one; }, c1);
        mf_layer<33, M::A2>(A, lane, [&](int st) { return st < 32 ? relu(c1[st >> 4][st & 15]) : one; }, c2);
        mf_layer<33, M::A3>(A, lane, [&](int st) { return st < 32 ? relu(c2[st >> 4][st & 15]) : one; }, c3);
        float part = 0.f;
#pragma unroll
        for (int q = 0; q < 32; ++q) part = fmaf(A[M::W4 + q * 64 + lane], relu(c3[q >> 4][q & 15]), part);
        const float out = b4 + (part + __shfl_xor(part, 32, 64));
        const long long r = t * 32 + (lane & 31);
        if (r < count && h == 0) top.insert(out, begin + r);
    }
    float* const ov = pv + (size_t)blockIdx.x * KMAX;
    long long* const oi = pi + (size_t)blockIdx.x * KMAX;
    block_topk(top, k, S, [&](int q, float v, long long i) {
        ov[q] = v;
        oi[q] = i;
    });
}

__global__ void __launch_bounds__(1024) k_sweep_final(const float* __restrict__ pv, const long long* __restrict__ pi,
                                                      int lists, int k, float* top_val, long long* top_idx) {
    __shared__ TopkLds<16> S;
    TopK top;
    top.init();
    for (int b = threadIdx.x; b < lists; b += 1024)
#pragma unroll
        for (int q = 0; q < KMAX; ++q)
            if (q < k) top.insert(pv[b * KMAX + q], pi[b * KMAX + q]);
    block_topk(top, k, S, [&](int q, float v, long long i) {
        top_val[q] = v;
        top_idx[q] = i;
    });
}

}  // namespace mlp

namespace mlp {

// Per-block top-k lists of the sweep: values, then (256-byte aligned) indices.
constexpr size_t sweep_scratch_bytes() {
    return (((size_t)SWEEP_MAXB * KMAX * sizeof(float) + 255) & ~(size_t)255) +
           (size_t)SWEEP_MAXB * KMAX * sizeof(long long);
}

// Device scratch of fv_mlp_sweep_static: room for the per-block lists of the
// largest sweep grid (SWEEP_MAXB blocks; larger counts are covered by the
// kernel's grid-stride loop, so no count needs more). Every device the
// library runs on holds its own copy until the process ends.
constexpr size_t STATIC_SCRATCH_BYTES = 393216;
static_assert(STATIC_SCRATCH_BYTES >= sweep_scratch_bytes(), "static sweep scratch too small");
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static std::mutex scratch_mu;
static void* scratch_ptr[MAX_DEVICES];

// Device address of `scratch` on the current device, looked up once per
// device (the host-side name of the array is not a device address).
static int static_scratch(void** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        fprintf(stderr, "fv_mlp_sweep_static: no usable current device\n");
        return FV_EDEVICE;
    }
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            fprintf(stderr, "fv_mlp_sweep_static: hipGetSymbolAddress failed: %s\n", hipGetErrorString(e));
            return FV_EDEVICE;
        }
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return FV_OK;
}

static int launch_status() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        fprintf(stderr, "fv_mlp: launch failed: %s\n", hipGetErrorString(e));
        return FV_EDEVICE;
    }
    return FV_OK;
}

// Validates the sweep's arguments and enqueues it with the per-block lists in
// `ws` (at least sweep_scratch_bytes(), 256-byte aligned). Every list entry
// the final selection reads is written by the block kernel of the same call,
// so `ws` needs no clearing.
static int sweep_launch(const float* params, const fv_tune_space* space, int64_t begin, int64_t count, int32_t k,
                        int64_t* top_idx, float* top_val, void* ws, hipStream_t st) {
    if (!params || !space || !top_idx || !top_val || !ws) return FV_EINVAL;
    if (k < 1 || k > KMAX || begin < 0 || count < 1) return FV_EINVAL;
    if (space->n_extra != 0 && space->n_extra != FV_MLP_MAX_EXTRA) return FV_EINVAL;
    SweepTab tab;
    int64_t total = 1;
    for (int s = 0; s < FV_NSITES; ++s) {
        const int r = space->radix[s];
        if (r < 1 || r > FV_SPACE_MAXC) return FV_EINVAL;
        tab.radix[s] = r;
        total *= r;
        for (int c = 0; c < FV_SPACE_MAXC; ++c) {
            tab.f[0][s][c] = c < r ? space->f1[s][c] : 0.f;
            tab.f[1][s][c] = c < r ? space->f2[s][c] : 0.f;
        }
    }
    for (int j = 0; j < FV_MLP_MAX_EXTRA; ++j) tab.extra[j] = j < space->n_extra ? space->extra[j] : 0.f;
    if (begin + count > total) return FV_EINVAL;
    // A workgroup's four waves take 32 configurations each per round. As many
    // workgroups as are resident (three a CU, by their LDS), so that the weights
    // are staged and the lists selected once a CU's place: 2M configurations take
    // 0.335 ms on 768 workgroups, 0.412 on 4096. Above 512 rounds a wave, more,
    // which even out the CUs' ends: 189M take 26.1 ms on 768, 25.9 on 4096.
    long long blocks = (count + 4 * 32 - 1) / (4 * 32);
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 0;
    const long long resident = 3LL * cus;
    const long long most = resident > 0 && resident < SWEEP_MAXB && blocks <= 512 * resident ? resident : SWEEP_MAXB;
    if (blocks > most) blocks = most;
    float* pv = (float*)ws;
    long long* pi = (long long*)((char*)ws + (((size_t)SWEEP_MAXB * KMAX * sizeof(float) + 255) & ~(size_t)255));
    if (space->n_extra == 0)
        hipLaunchKernelGGL(k_sweep_mfma<FV_MLP_IN>, dim3((unsigned)blocks), dim3(SWEEP_T), 0, st, params, tab,
                           (long long)begin, (long long)count, k, pv, pi);
    else
        hipLaunchKernelGGL(k_sweep_mfma<FV_MLP_IN_SIZED>, dim3((unsigned)blocks), dim3(SWEEP_T), 0, st, params, tab,
                           (long long)begin, (long long)count, k, pv, pi);
    hipLaunchKernelGGL(k_sweep_final, dim3(1), dim3(1024), 0, st, pv, pi, (int)blocks, k, top_val,
                       (long long*)top_idx);
    return launch_status();
}

}  // namespace mlp

// ---------------------------------------------------------------------------
// C ABI.

static int mlp_check_launch() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        fprintf(stderr, "fv_mlp: launch failed: %s\n", hipGetErrorString(e));
        return FV_EDEVICE;
    }
    return FV_OK;
}

extern "C" {

int fv_mlp_workspace(int32_t n, size_t* bytes) {
    if (n < 1 || n > mlp::MAXN || !bytes) return FV_EINVAL;
    *bytes = mlp::scratch_bytes(n);
    return FV_OK;
}

int fv_mlp_loss_grad(const float* params, int32_t n_in, const float* X, const float* y, int32_t n, float alpha,
                     float* grad, float* loss, void* workspace, size_t ws_bytes, void* stream) {
    if (!params || !X || !y || !grad || !loss || !workspace) return FV_EINVAL;
    if (n_in != FV_MLP_IN && n_in != FV_MLP_IN_SIZED) return FV_EINVAL;
    if (n < 1 || n > mlp::MAXN || !(alpha >= 0.f)) return FV_EINVAL;
    if (ws_bytes < mlp::scratch_bytes(n)) return FV_EWORKSPACE;
    if (n_in == FV_MLP_IN)
        hipLaunchKernelGGL(mlp::k_loss_grad<FV_MLP_IN>, dim3(1), dim3(mlp::TT), 0, (hipStream_t)stream, params, X, y,
                           n, alpha, grad, loss);
    else
        hipLaunchKernelGGL(mlp::k_loss_grad<FV_MLP_IN_SIZED>, dim3(1), dim3(mlp::TT), 0, (hipStream_t)stream, params,
                           X, y, n, alpha, grad, loss);
    return mlp_check_launch();
}

int fv_mlp_predict(const float* params, int32_t n_in, const float* X, int32_t n, float* out, void* stream) {
    if (!params || !X || !out || n < 0) return FV_EINVAL;
    if (n_in != FV_MLP_IN && n_in != FV_MLP_IN_SIZED) return FV_EINVAL;
    if (n == 0) return FV_OK;
    if (n_in == FV_MLP_IN)
        hipLaunchKernelGGL(mlp::k_predict<FV_MLP_IN>, dim3((n + 127) / 128), dim3(mlp::SWEEP_T), 0,
                           (hipStream_t)stream, params, X, n, out);
    else
        hipLaunchKernelGGL(mlp::k_predict<FV_MLP_IN_SIZED>, dim3((n + 127) / 128), dim3(mlp::SWEEP_T), 0,
                           (hipStream_t)stream, params, X, n, out);
    return mlp_check_launch();
}

int fv_mlp_train_bounded(float* params, int32_t n_in, float* adam_m, float* adam_v, int32_t* adam_t, const float* X,
                         const float* y, int32_t n, const int32_t* order, const fv_mlp_hparams* hp, float* epoch_loss,
                         int32_t* epochs_run, void* workspace, size_t ws_bytes, int32_t roll_polls, int32_t wait_polls,
                         void* stream) {
    if (!params || !adam_m || !adam_v || !adam_t || !X || !y || !order || !hp || !epoch_loss || !epochs_run ||
        !workspace || roll_polls < 0 || wait_polls < 0)
        return FV_EINVAL;
    if (n_in != FV_MLP_IN && n_in != FV_MLP_IN_SIZED) return FV_EINVAL;
    if (n < 1 || n > mlp::MAXN || hp->batch < 1 || hp->max_epochs < 0 || hp->n_iter_no_change < 0) return FV_EINVAL;
    if (!(hp->lr > 0.f) || !(hp->beta1 >= 0.f && hp->beta1 < 1.f) || !(hp->beta2 >= 0.f && hp->beta2 < 1.f) ||
        !(hp->eps > 0.f) || !(hp->alpha >= 0.f))
        return FV_EINVAL;
    const int bmax = hp->batch < n ? hp->batch : n;
    if (ws_bytes < mlp::scratch_bytes(bmax)) return FV_EWORKSPACE;
    const int wgs = mlp::train_workgroups(bmax, (hipStream_t)stream);
    char* const ex = (char*)(((uintptr_t)workspace + 63) & ~(uintptr_t)63);
    if (wgs > 1) hipLaunchKernelGGL(mlp::k_train_clear, dim3(1), dim3(64), 0, (hipStream_t)stream, (unsigned*)ex);
#define FV_TRAIN(IN, ALONE, GRID)                                                                                 \
    hipLaunchKernelGGL((mlp::k_train<IN, ALONE>), dim3(GRID), dim3(mlp::TT), 0, (hipStream_t)stream, params,       \
                       adam_m, adam_v, adam_t, X, y, n, order, *hp, epoch_loss, epochs_run, ex, wgs, roll_polls, \
                       wait_polls)
    if (n_in == FV_MLP_IN) {
        FV_TRAIN(FV_MLP_IN, false, wgs);
        if (wgs > 1) FV_TRAIN(FV_MLP_IN, true, 1);
    } else {
        FV_TRAIN(FV_MLP_IN_SIZED, false, wgs);
        if (wgs > 1) FV_TRAIN(FV_MLP_IN_SIZED, true, 1);
    }
#undef FV_TRAIN
    return mlp_check_launch();
}

int fv_mlp_train(float* params, int32_t n_in, float* adam_m, float* adam_v, int32_t* adam_t, const float* X,
                 const float* y, int32_t n, const int32_t* order, const fv_mlp_hparams* hp, float* epoch_loss,
                 int32_t* epochs_run, void* workspace, size_t ws_bytes, void* stream) {
    return fv_mlp_train_bounded(params, n_in, adam_m, adam_v, adam_t, X, y, n, order, hp, epoch_loss, epochs_run,
                                workspace, ws_bytes, mlp::ROLL_POLLS, mlp::WAIT_POLLS, stream);
}

int fv_mlp_sweep_workspace(size_t* bytes) {
    if (!bytes) return FV_EINVAL;
    *bytes = mlp::sweep_scratch_bytes();
    return FV_OK;
}

int fv_mlp_sweep(const float* params, const fv_tune_space* space, int64_t begin, int64_t count, int32_t k,
                 int64_t* top_idx, float* top_val, void* workspace, size_t ws_bytes, void* stream) {
    if (!workspace) return FV_EINVAL;
    if (ws_bytes < mlp::sweep_scratch_bytes()) return FV_EWORKSPACE;
    return mlp::sweep_launch(params, space, begin, count, k, top_idx, top_val, workspace, (hipStream_t)stream);
}

int fv_mlp_sweep_static(const float* params, const fv_tune_space* space, int64_t begin, int64_t count, int32_t k,
                        int64_t* top_idx, float* top_val, void* stream) {
    // Sizes: k above 8 is rejected by the argument check (FV_EINVAL); any
    // count fits, the block count being capped at the scratch's capacity.
    void* ws = nullptr;
    const int rc = mlp::static_scratch(&ws);
    if (rc != FV_OK) return rc;
    return mlp::sweep_launch(params, space, begin, count, k, top_idx, top_val, ws, (hipStream_t)stream);
}

}  // extern "C"
