// The learned start-value proposal: a 1024-256-256-4 perceptron that maps
// the residual patch around the peak to the start point of the new
// component's fit, in place of the simple initial values of Sect. 3 (the
// residual peak and the main-lobe width).  The LM fit of Sect. 3 runs from the
// proposal and decides whether it is kept: when that fit does not converge,
// or ends with a new component of amplitude zero, the fit kernel fits the
// simple values instead.
//
// Network: h1 = relu(W1 x + b1), h2 = relu(W2 h1 + b2), y = W3 h2 + b3.
//   x = the 32 x 32 patch around the peak pixel (r*, c*), rows r*-16..r*+15,
//       columns c*-16..c*+15, zero outside the image, divided by R[p*];
//   y = (a / R[p*], log(s / omega_b), x - c*, y - r*) of the fitted new
//       component (convolved space, before the loop gain).
// Flat parameter order: W1 (256 x 1024, row-major), b1, W2 (256 x 256), b2,
// W3 (4 x 256), b3; 329220 FP32 values.
//
// This file holds
//   * the inference kernel of the minor cycle (64 work-groups, which also
//     record the patch of (patch, target) training pairs when asked),
//   * the training kernels: FP32 products on the matrix cores with fused row
//     gather and bias / ReLU / ReLU mask epilogues, the output layer with the
//     MSE gradient, column sums and Adam; the forward pass over many rows,
//   * the trainer object of the C ABI (asp_mlp_*).
// The training loss is the mean over samples and outputs of (y - t)^2.
#include <math.h>
#include <string.h>

#include <string>

#include "asp_device.h"

namespace asp {

// ===========================================================================
// Inference inside the minor cycle.
// ===========================================================================

constexpr int kPT = 256;                          // threads per work-group
constexpr int kUnits = kNetH / kPropGroups;       // first-layer units per work-group
constexpr int kPerThread = kNetIn / kPT;          // patch inputs per thread
static_assert(kNetH == kPT, "one thread per second-layer unit");
static_assert(kNetOut * 64 == kPT, "one wave per output");
static_assert(kUnits * kPropGroups == kNetH && kUnits == 4, "four first-layer units per group");
static_assert(kPerThread == 4 && kPatch % kPerThread == 0, "four inputs of one patch row");

// The peak pixel of this iteration (the forced index of a caller's fit, else
// the decoded peak key) and the residual there; false when there is none (the
// fit kernel reports that state) or after a stop.  The stop flag, the forced
// index and the key slots are read in one round trip.  Every thread of the
// work-group calls it.
__device__ inline bool proposal_centre(const Params &p, unsigned long long *key_s, int64_t *r0,
                                       int64_t *c0, float *v)
{
    DevState *st = p.st;
    const int32_t stop = st->stop;
    int64_t idx = st->forced_idx;
    const unsigned long long key = collect_peak_key(st, false, key_s);
    if (stop) return false;
    if (idx < 0) {
        if (key == 0ull) return false;
        idx = (int64_t)(0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull));
    }
    if (idx >= p.H * p.W) return false;
    *r0 = idx / p.W;
    *c0 = idx % p.W;
    *v = p.R[idx];
    return true;
}

// One launch of kPropGroups work-groups.  Work-group g:
//   * gathers the whole patch (thread t holds inputs 4t .. 4t+3, four
//     neighbours of one patch row) and, when the context collects training
//     pairs, records inputs 16g .. 16g+15;
//   * forms first-layer units 4g .. 4g+3 completely (per-thread products,
//     then a fixed-order reduction over lanes and waves);
//   * writes the contribution of those four units to every second-layer
//     pre-activation (thread u: unit u), one row of the partial-sum scratch.
// The work-group that arrives last adds the rows in work-group order, applies
// the bias and ReLU, runs the output layer and writes the proposal.  Every
// load that does not depend on another is issued at the start.  Without a
// peak, or after a stop, every work-group leaves before the arrival, so the
// counter stays a multiple of the grid.
__global__ __launch_bounds__(kPT) void k_propose(Params p, NetParams net, int use_net)
{
    DevState *st = p.st;
    __shared__ float red[kPT / 64][kUnits];
    __shared__ float h1[kUnits];
    __shared__ float h2[kNetH];
    __shared__ float outs[kNetOut];
    __shared__ unsigned long long key_s;
    __shared__ int last_s;
    const int t = threadIdx.x, g = blockIdx.x;
    const int wave = t >> 6, lane = t & 63;
    float4 w1[kUnits];
    float w2[kUnits], w3[kNetH / 64];
    float b1 = 0.0f, b2 = 0.0f, b3 = 0.0f;
    if (use_net) {
#pragma unroll
        for (int j = 0; j < kUnits; ++j)
            w1[j] = *reinterpret_cast<const float4 *>(net.w1 + (int64_t)(g * kUnits + j) * kNetIn +
                                                      kPerThread * t);
#pragma unroll
        for (int j = 0; j < kUnits; ++j) w2[j] = net.w2t[(g * kUnits + j) * kNetH + t];
#pragma unroll
        for (int i = 0; i < kNetH / 64; ++i) w3[i] = net.w3[wave * kNetH + lane + 64 * i];
        b1 = t < kUnits ? net.b1[g * kUnits + t] : 0.0f;
        b2 = net.b2[t];
        b3 = lane == 0 ? net.b3[wave] : 0.0f;
    }
    int64_t r0, c0;
    float v;
    if (!proposal_centre(p, &key_s, &r0, &c0, &v)) return;
    float x[kPerThread];
    {
        const int e0 = kPerThread * t;
        const int64_t r = r0 - kPatchHalf + e0 / kPatch;
        const int64_t cb = c0 - kPatchHalf + e0 % kPatch;
        const bool row_in = r >= 0 && r < p.H;
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const int64_t c = cb + i;
            x[i] = (row_in && c >= 0 && c < p.W) ? p.R[r * p.W + c] / v : 0.0f;
        }
        if (p.rec_cap > 0 && (e0 >> 4) == g && st->rec_n < p.rec_cap) {
            float *rp = p.rec_patch + st->rec_n * kNetIn + e0;
#pragma unroll
            for (int i = 0; i < kPerThread; ++i) rp[i] = x[i];
        }
    }
    if (!use_net) return;
    // first layer: units 4g .. 4g+3
    {
        float acc[kUnits];
#pragma unroll
        for (int j = 0; j < kUnits; ++j)
            acc[j] = w1[j].x * x[0] + w1[j].y * x[1] + w1[j].z * x[2] + w1[j].w * x[3];
#pragma unroll
        for (int j = 0; j < kUnits; ++j)
            for (int off = 32; off > 0; off >>= 1) acc[j] += __shfl_xor(acc[j], off, 64);
        if (lane < kUnits) {
            float a = acc[0];
#pragma unroll
            for (int j = 1; j < kUnits; ++j) a = lane == j ? acc[j] : a;
            red[wave][lane] = a;
        }
        __syncthreads();
        if (t < kUnits) {
            float a = b1;
#pragma unroll
            for (int q = 0; q < kPT / 64; ++q) a += red[q][t];
            h1[t] = a > 0.0f ? a : 0.0f;
        }
        __syncthreads();
    }
    // this group's share of every second-layer pre-activation
    {
        float a = 0.0f;
#pragma unroll
        for (int j = 0; j < kUnits; ++j) a += w2[j] * h1[j];
        net.part[g * kNetH + t] = a;
    }
    // arrival: the barrier orders every thread's stores before thread 0's
    // release; the last arrival's acquire pairs with the others' releases
    __syncthreads();
    if (t == 0) {
        const unsigned int before = __hip_atomic_fetch_add(net.done, 1u, __ATOMIC_ACQ_REL,
                                                           __HIP_MEMORY_SCOPE_AGENT);
        last_s = (before + 1u) % kPropGroups == 0u ? 1 : 0;
    }
    __syncthreads();
    if (!last_s) return;
    {
        float part[kPropGroups];
#pragma unroll
        for (int q = 0; q < kPropGroups; ++q)
            part[q] = __hip_atomic_load(&net.part[q * kNetH + t], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
        float a = b2;
#pragma unroll
        for (int q = 0; q < kPropGroups; ++q) a += part[q];
        h2[t] = a > 0.0f ? a : 0.0f;
    }
    __syncthreads();
    {
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < kNetH / 64; ++i) a += w3[i] * h2[lane + 64 * i];
        for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
        if (lane == 0) outs[wave] = a + b3;
    }
    __syncthreads();
    if (t == 0) {
        const double vv = (double)v;
        st->proposal[0] = (double)outs[0] * vv;
        st->proposal[1] = (double)c0 + (double)outs[2];
        st->proposal[2] = (double)r0 + (double)outs[3];
        st->proposal[3] = st->omega_b * exp((double)outs[1]);
        st->have_proposal = 2;
    }
}

hipError_t launch_propose(const Params &p, const NetParams &net, int use_net, hipStream_t s)
{
    hipLaunchKernelGGL(k_propose, dim3(kPropGroups), dim3(kPT), 0, s, p, net, use_net);
    return hipGetLastError();
}

// ===========================================================================
// Training kernels.
// ===========================================================================

// Every product C[m][n] = sum_k A(m, k) B(k, n) runs on v_mfma_f32_16x16x4f32,
// which adds its four products one after another in order of k, each with one
// rounding: a chain of these instructions over k is the chain of scalar FMAs in
// order of k, bit for bit (checked against it, tiny values included).  The sum
// over k is not split, so a wave's 16 x 16 tile is one dependent chain of K / 4
// instructions of 32 clocks and a product's time is bound by that chain while
// there are fewer tiles than SIMDs (3.4 us at K = 1024); the tiles are
// therefore the smallest the instruction has.  A step of 512 rows takes six
// launches, 72 us; with 64 x 64 tiles of scalar FMAs, a copy of the picked rows
// and column sums by one thread a column it took fifteen and 857 us.

typedef float f32x4 __attribute__((ext_vector_type(4)));

// A row-major operand: rows x cols at stride ld, the rows picked by idx when
// given (an index outside [0, n_src) reads as a row of zeros and sets *bad).
// cols is a multiple of 4.
struct Op {
    const float *p;
    int64_t ld;
    int rows, cols;
    const int32_t *idx;
    int64_t n_src;
    int32_t *bad;
    int vec;                       // rows start on 16 bytes
};

// Where row `row` starts, from p; -1 for a row of zeros.
__device__ __forceinline__ int64_t row_offset(const Op &a, int row, int picked)
{
    if (row >= a.rows) return -1;
    if (!a.idx) return row * a.ld;
    if (picked < 0 || picked >= a.n_src) {
        *a.bad = 1;
        return -1;
    }
    return picked * a.ld;
}

__device__ __forceinline__ f32x4 load4(const Op &a, int64_t off, int col)
{
    if (off < 0 || col >= a.cols) return f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float *q = a.p + off + col;
    if (a.vec) return *reinterpret_cast<const f32x4 *>(q);
    return f32x4{q[0], q[1], q[2], q[3]};
}

// 32 x 32 output tile of a 256-thread work-group, one 16 x 16 tile per wave.
// An operand is contiguous along k (KMajor: rows are m or n) or along m / n
// (rows are k).  kKC values of k at a time go through LDS, two buffers; kAhead
// chunks are on their way in registers, as a wave works through one in 16
// instructions, 0.21 us, and a load from memory takes longer.  The row strides
// in LDS (kKC + 4 and 48 floats) put the 16 x 4 values of one instruction's
// operand into 64 different banks.
constexpr int kTile = 32, kKC = 64, kAhead = 8;
constexpr int kStrideK = kKC + 4, kStrideM = 48;
constexpr int kBufFloats = kKC * kStrideM;              // the larger of the two layouts
static_assert(kTile * kStrideK <= kBufFloats, "operand buffer");
constexpr size_t kGemmLds = sizeof(float) * 4 * kBufFloats;
constexpr int kLoads = kTile * kKC / 4 / 256;           // f32x4 per thread, operand and chunk

// A thread's share of an operand, chunk after chunk.
template <bool KMajor>
struct Loader {
    const Op &a;
    int o0;
    int64_t off[kLoads];           // KMajor: its rows
    int32_t pick[kLoads];          // else: the index of its rows of the next chunk

    static __device__ int row(int u) { return (threadIdx.x + 256 * u) / (KMajor ? kKC / 4 : kTile / 4); }
    static __device__ int col() { return 4 * (threadIdx.x % (KMajor ? kKC / 4 : kTile / 4)); }

    __device__ __forceinline__ void picks(int r0)
    {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const int r = r0 + row(u);
            pick[u] = a.idx && r < a.rows ? a.idx[r] : 0;
        }
    }
    __device__ __forceinline__ Loader(const Op &op, int start) : a(op), o0(start)
    {
        picks(KMajor ? o0 : 0);
        if (KMajor) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u) off[u] = row_offset(a, o0 + row(u), pick[u]);
        }
    }
    __device__ __forceinline__ void fetch(int k0, f32x4 (&v)[kLoads])
    {
        if (!KMajor) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u) off[u] = row_offset(a, k0 + row(u), pick[u]);
            if (a.idx) picks(k0 + kKC);
        }
#pragma unroll
        for (int u = 0; u < kLoads; ++u) v[u] = load4(a, off[u], KMajor ? k0 + col() : o0 + col());
    }
};

template <bool KMajor>
__device__ __forceinline__ void stage(float *buf, const f32x4 (&v)[kLoads])
{
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        const int e = threadIdx.x + 256 * u;
        float *q = KMajor ? buf + (e / (kKC / 4)) * kStrideK + 4 * (e % (kKC / 4))
                          : buf + (e / (kTile / 4)) * kStrideM + 4 * (e % (kTile / 4));
        *reinterpret_cast<f32x4 *>(q) = v[u];
    }
}

// Lane l of a wave ends with rows 4 (l / 16) + r, r < 4, of column l % 16.
// With Ones every B(k, n) is 1: the sums over k of A, in order.
template <bool AK, bool BK, bool Ones = false>
__device__ __forceinline__ f32x4 product(const Op &A, const Op &B, int m0, int n0, int K, float *lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int mi = 16 * (wave >> 1) + i, ni = 16 * (wave & 1) + i;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 va[kAhead][kLoads], vb[kAhead][kLoads];
    Loader<AK> fa(A, m0);
    Loader<BK> fb(B, n0);
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
        if (d * kKC < K) {
            fa.fetch(d * kKC, va[d]);
            if (!Ones) fb.fetch(d * kKC, vb[d]);
        }
    }
    for (int k1 = 0; k1 < K; k1 += kAhead * kKC) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
            const int k0 = k1 + d * kKC;
            if (k0 >= K) break;
            float *la = lds + 2 * (d & 1) * kBufFloats, *lb = la + kBufFloats;
            stage<AK>(la, va[d]);
            if (!Ones) stage<BK>(lb, vb[d]);
            __syncthreads();               // also: the other buffers have been read
            if (k0 + kAhead * kKC < K) {
                fa.fetch(k0 + kAhead * kKC, va[d]);
                if (!Ones) fb.fetch(k0 + kAhead * kKC, vb[d]);
            }
            const float *pa = AK ? la + mi * kStrideK + g : la + g * kStrideM + mi;
            const float *pb = BK ? lb + ni * kStrideK + g : lb + g * kStrideM + ni;
            const int steps = K - k0 < kKC ? (K - k0 + 3) / 4 : kKC / 4;
            auto step = [&](int q) __attribute__((always_inline)) {
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    pa[AK ? 4 * q : 4 * q * kStrideM],
                    Ones ? 1.0f : pb[BK ? 4 * q : 4 * q * kStrideM], acc, 0, 0, 0);
            };
            if (steps == kKC / 4) {
#pragma unroll
                for (int q = 0; q < kKC / 4; ++q) step(q);
            } else {
                for (int q = 0; q < steps; ++q) step(q);     // past K the operands are zeros
            }
        }
    }
    return acc;
}

// The tile's epilogue and store: bias with ReLU (bias given), or the ReLU
// derivative (mask given: 0 where mask <= 0), or neither.
__device__ __forceinline__ void store_tile(const f32x4 &acc, int m0, int n0, int M, int N, float *C,
                                           const float *bias, const float *mask)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = n0 + 16 * (wave & 1) + (lane & 15);
    if (n >= N) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + 16 * (wave >> 1) + 4 * (lane >> 4) + r;
        if (m >= M) continue;
        const int64_t o = (int64_t)m * N + n;
        float v = acc[r];
        if (bias) {
            v += bias[n];
            v = v > 0.0f ? v : 0.0f;
        }
        if (mask) v = mask[o] > 0.0f ? v : 0.0f;
        C[o] = v;
    }
}

// A hidden layer: out = relu(X W^T + b), X M x K (rows by idx), W N x K.
__global__ __launch_bounds__(256) void k_layer(Op X, Op W, const float *bias, float *out)
{
    extern __shared__ __align__(16) float lds[];
    const int m0 = blockIdx.y * kTile, n0 = blockIdx.x * kTile;
    const f32x4 acc = product<true, true>(X, W, m0, n0, X.cols, lds);
    store_tile(acc, m0, n0, X.rows, W.rows, out, bias, nullptr);
}

// The output layer, sixteen rows per work-group: Y = H2 W3^T + b3.  Loss: not Y but
// dY = 2 (Y - T) / (B d), these rows' sum of (Y - T)^2 in FP64 and
// dH2 = (dY W3) * [H2 > 0]; T's rows are picked by idx.  The first wave has the
// chain of products, the others share the loads and dH2.
constexpr int kHeadRows = 16;
template <bool Loss>
__global__ __launch_bounds__(256) void k_head(const float *H2, const float *w3, const float *b3, Op T,
                                             float *dY, float *dH2, double *part)
{
    __shared__ __align__(16) float h[kHeadRows][kNetH + 4], w[kNetOut][kNetH + 4];
    __shared__ float d[kHeadRows][kNetOut + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
    const int m0 = blockIdx.x * kHeadRows, M = T.rows;
    static_assert(kNetH == 256 && kNetOut == 4, "a wave reads a row of W3 and four of H2");
    f32x4 v[4];
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int32_t pick[4] = {0, 0, 0, 0};
    if (Loss && T.idx && wave == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (m0 + 4 * g + r < M) pick[r] = T.idx[m0 + 4 * g + r];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int m = m0 + 4 * wave + u;
        v[u] = m < M ? *reinterpret_cast<const f32x4 *>(H2 + (int64_t)m * kNetH + 4 * lane)
                     : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    const f32x4 vw = *reinterpret_cast<const f32x4 *>(w3 + wave * kNetH + 4 * lane);
    if (Loss && wave == 0 && i < kNetOut) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t off = row_offset(T, m0 + 4 * g + r, pick[r]);
            if (off >= 0) t[r] = T.p[off + i];
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) *reinterpret_cast<f32x4 *>(&h[4 * wave + u][4 * lane]) = v[u];
    *reinterpret_cast<f32x4 *>(&w[wave][4 * lane]) = vw;
    __syncthreads();
    if (wave == 0) {
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 16
        for (int q = 0; q < kNetH / 4; ++q) {
            const float b = w[i & 3][4 * q + g];
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(h[i][4 * q + g], i < kNetOut ? b : 0.0f, acc, 0, 0, 0);
        }
        const float scale = 2.0f / (float)(M * kNetOut);
        double s = 0.0;
        if (i < kNetOut) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + 4 * g + r;
                const float y = acc[r] + b3[i];
                float e = 0.0f;
                if (m < M) {
                    if (Loss) {
                        const float diff = y - t[r];
                        e = scale * diff;
                        s += (double)diff * (double)diff;
                    }
                    dY[(int64_t)m * kNetOut + i] = Loss ? e : y;
                }
                d[4 * g + r][i] = e;
            }
        }
        if (Loss) {
            for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            if (lane == 0) part[blockIdx.x] = s;
        }
    }
    if (!Loss) return;
    __syncthreads();
    const float a = d[i][g];
#pragma unroll
    for (int u = 0; u < kNetH / 64; ++u) {
        const int n = 64 * wave + 16 * u + i;
        const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
        const f32x4 o = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w[g][n], z, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + 4 * g + r;
            if (m < M) dH2[(int64_t)m * kNetH + n] = h[4 * g + r][n] > 0.0f ? o[r] : 0.0f;
        }
    }
}

// out[n] = sum over m of X(m, n) for n0 <= n < n0 + 32, in row order (the bias
// gradients).
__device__ __forceinline__ void column_sums(const Op &X, int n0, float *out, float *lds)
{
    const f32x4 acc = product<false, false, true>(X, X, n0, 0, X.rows, lds);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((wave & 1) || (lane & 15)) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int n = n0 + 16 * (wave >> 1) + 4 * (lane >> 4) + r;
        if (n < X.cols) out[n] = acc[r];
    }
}

// What the output layer's gradient allows, in one launch: the tiles of
// dH1 = (dH2 W2) * [H1 > 0], of dW2 = dH2^T H1 and of dW3 = dY^T H2, and the
// column sums db2 and db3.
struct Back {
    int M;
    const float *dY, *H1, *H2, *w2;
    float *dH2, *dH1, *dw2, *db2, *dw3, *db3;
};
constexpr int kHTiles = kNetH / kTile;

__global__ __launch_bounds__(256) void k_back(Back b)
{
    extern __shared__ __align__(16) float lds[];
    const int M = b.M, mt = (M + kTile - 1) / kTile;
    int t = blockIdx.x;
    const Op dH2{b.dH2, kNetH, M, kNetH, nullptr, 0, nullptr, 1};
    // the longest first: dW2 and dW3 run over the rows
    if (t < kHTiles * kHTiles) {
        const int m0 = (t / kHTiles) * kTile, n0 = (t % kHTiles) * kTile;
        const Op H1{b.H1, kNetH, M, kNetH, nullptr, 0, nullptr, 1};
        const f32x4 acc = product<false, false>(dH2, H1, m0, n0, M, lds);
        store_tile(acc, m0, n0, kNetH, kNetH, b.dw2, nullptr, nullptr);
        return;
    }
    t -= kHTiles * kHTiles;
    if (t < kHTiles) {
        const int n0 = t * kTile;
        const Op dY{b.dY, kNetOut, M, kNetOut, nullptr, 0, nullptr, 1};
        const Op H2{b.H2, kNetH, M, kNetH, nullptr, 0, nullptr, 1};
        const f32x4 acc = product<false, false>(dY, H2, 0, n0, M, lds);
        store_tile(acc, 0, n0, kNetOut, kNetH, b.dw3, nullptr, nullptr);
        return;
    }
    t -= kHTiles;
    if (t <= kHTiles) {
        const Op dY{b.dY, kNetOut, M, kNetOut, nullptr, 0, nullptr, 1};
        if (t < kHTiles) column_sums(dH2, t * kTile, b.db2, lds);
        else column_sums(dY, 0, b.db3, lds);
        return;
    }
    t -= kHTiles + 1;
    if (t < kHTiles * mt) {
        const int m0 = (t / kHTiles) * kTile, n0 = (t % kHTiles) * kTile;
        const Op W2{b.w2, kNetH, kNetH, kNetH, nullptr, 0, nullptr, 1};
        const f32x4 acc = product<true, false>(dH2, W2, m0, n0, kNetH, lds);
        store_tile(acc, m0, n0, M, kNetH, b.dH1, nullptr, b.H1);
    }
}
constexpr int kBackFixed = kHTiles * kHTiles + 2 * kHTiles + 1;

// dW1 = dH1^T X, db1, and the batch loss sum((Y - T)^2) / (B d) added to *loss.
__global__ __launch_bounds__(256) void k_back1(Op X, const float *dH1, float *dw1, float *db1,
                                               const double *part, int n_part, double *loss)
{
    extern __shared__ __align__(16) float lds[];
    constexpr int NT = kNetIn / kTile;
    const int M = X.rows, t = blockIdx.x;
    const Op dH{dH1, kNetH, M, kNetH, nullptr, 0, nullptr, 1};
    if (t < kHTiles * NT) {
        const int m0 = (t / NT) * kTile, n0 = (t % NT) * kTile;
        const f32x4 acc = product<false, false>(dH, X, m0, n0, M, lds);
        store_tile(acc, m0, n0, kNetH, kNetIn, dw1, nullptr, nullptr);
    } else if (t < kHTiles * (NT + 1)) {
        column_sums(dH, (t - kHTiles * NT) * kTile, db1, lds);
    } else {
        // one work-group, fixed summation order
        double *red = reinterpret_cast<double *>(lds);
        double s = 0.0;
        for (int i = threadIdx.x; i < n_part; i += 256) s += part[i];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss += red[0] / (double)(M * kNetOut);
    }
}

// The forward pass over many rows in one launch: a work-group per CU with an
// even share of the tiles of sixteen rows, up to kRT of them at a time through
// all three layers with the hidden values in LDS, wave w the columns
// 32 w .. 32 w + 31 of a layer, RT x 2 tiles of 16 x 16.  The weights (1.3 MB,
// from L2, once per kRT tiles) and X stream through LDS kFC values of k at a
// time, two buffers and kFAhead chunks on their way.  The bound is the matrix
// cores at 256 FP32 flops a clock and CU: 50000 rows take 350 us, 61 % of that
// rate (layer by layer with 512 rows a launch they took 25 ms).  32 rows a
// work-group, two work-groups a CU, took 405 us: twice the reads of the weights.
constexpr int kFC = 16, kFAhead = 4, kFStride = kFC + 4, kHStride = kNetH + 4, kRT = 4;
constexpr int kRowThreads = 512;
constexpr size_t kRowsLds =
    sizeof(float) * (2 * kNetH * kFStride + 2 * 16 * kRT * kFStride + 16 * kRT * kHStride);
static_assert(kNetIn % (kFC * kFAhead) == 0 && kNetH % (kFC * kFAhead) == 0 && kFAhead % 2 == 0, "chunks");
static_assert(kNetH == 32 * (kRowThreads / 64), "a wave has 32 columns");

struct Net {
    const float *w1, *b1, *w2, *b2, *w3, *b3;
};

// One hidden layer of 16 RT rows from X (FromX) or h into h.
template <int RT, bool FromX>
__device__ __forceinline__ void rows_layer(const Op &X, int m0, const float *W, const float *bias,
                                           float *wbuf, float *xbuf, float *h)
{
    constexpr int ROWS = 16 * RT, K = FromX ? kNetIn : kNetH, QC = kFC / 4;
    constexpr int WL = kNetH * QC / kRowThreads, WR = kRowThreads / QC;
    static_assert(ROWS <= WR, "one load of X per thread");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, i = lane & 15, g = lane >> 4;
    const int lr = t / QC, lc = 4 * (t % QC);              // this thread's row and column of a chunk
    const float *wp = W + (int64_t)lr * K + lc;
    const int64_t xo = FromX && lr < ROWS ? row_offset(X, m0 + lr, 0) : -1;
    f32x4 acc[RT][2], vw[kFAhead][WL], vx[kFAhead];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[r][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto fetch = [&](int d, int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < WL; ++u) vw[d][u] = *reinterpret_cast<const f32x4 *>(wp + u * WR * K + k0);
        if (FromX) vx[d] = load4(X, xo, k0 + lc);
    };
#pragma unroll
    for (int d = 0; d < kFAhead; ++d) fetch(d, d * kFC);
    for (int k1 = 0; k1 < K; k1 += kFAhead * kFC) {
#pragma unroll
        for (int d = 0; d < kFAhead; ++d) {
            const int k0 = k1 + d * kFC;
            float *wb = wbuf + (d & 1) * kNetH * kFStride, *xb = xbuf + (d & 1) * 16 * kRT * kFStride;
#pragma unroll
            for (int u = 0; u < WL; ++u) *reinterpret_cast<f32x4 *>(wb + (lr + u * WR) * kFStride + lc) = vw[d][u];
            if (FromX && lr < ROWS) *reinterpret_cast<f32x4 *>(xb + lr * kFStride + lc) = vx[d];
            __syncthreads();               // also: the other buffers have been read
            if (k0 + kFAhead * kFC < K) fetch(d, k0 + kFAhead * kFC);
            const float *pa = FromX ? xb + i * kFStride + g : h + i * kHStride + k0 + g;
            constexpr int RA = 16 * (FromX ? kFStride : kHStride);
            const float *pb = wb + (32 * wave + i) * kFStride + g;
#pragma unroll
            for (int q = 0; q < QC; ++q) {
                float xa[RT], xw[2];
#pragma unroll
                for (int r = 0; r < RT; ++r) xa[r] = pa[r * RA + 4 * q];
#pragma unroll
                for (int n = 0; n < 2; ++n) xw[n] = pb[16 * n * kFStride + 4 * q];
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int n = 0; n < 2; ++n)
                        acc[r][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[r], xw[n], acc[r][n], 0, 0, 0);
            }
        }
    }
    __syncthreads();                       // h and the buffers have been read
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int col = 32 * wave + 16 * n + i;
        const float b = bias[col];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float v = acc[r][n][q] + b;
                h[(16 * r + 4 * g + q) * kHStride + col] = v > 0.0f ? v : 0.0f;
            }
    }
    __syncthreads();
}

template <int RT>
__device__ __forceinline__ void rows_block(const Op &X, int m0, const Net &net, float *Y, float *lds)
{
    float *wbuf = lds;                                   // 2 x 256 x kFStride
    float *xbuf = wbuf + 2 * kNetH * kFStride;           // 2 x 16 kRT x kFStride
    float *h = xbuf + 2 * 16 * kRT * kFStride;           // 16 kRT x kHStride
    rows_layer<RT, true>(X, m0, net.w1, net.b1, wbuf, xbuf, h);
    rows_layer<RT, false>(X, m0, net.w2, net.b2, wbuf, xbuf, h);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, i = lane & 15, g = lane >> 4;
    if (t < kNetOut * kNetH / 4)
        *reinterpret_cast<f32x4 *>(wbuf + (t / (kNetH / 4)) * kHStride + 4 * (t % (kNetH / 4))) =
            *reinterpret_cast<const f32x4 *>(net.w3 + 4 * t);
    __syncthreads();
    // the output layer: wave r takes row tile r
    if (wave < RT) {
        const float *pa = h + (16 * wave + i) * kHStride + g, *pb = wbuf + (i & 3) * kHStride + g;
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 16
        for (int q = 0; q < kNetH / 4; ++q) {
            const float b = pb[4 * q];
            o = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[4 * q], i < kNetOut ? b : 0.0f, o, 0, 0, 0);
        }
        if (i < kNetOut) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = m0 + 16 * wave + 4 * g + q;
                if (m < X.rows) Y[(int64_t)m * kNetOut + i] = o[q] + net.b3[i];
            }
        }
    }
    __syncthreads();                       // the next rows overwrite h and wbuf
}

__global__ __launch_bounds__(kRowThreads) void k_rows(Op X, Net net, float *Y)
{
    extern __shared__ __align__(16) float lds[];
    const int64_t tiles = (X.rows + 15) / 16;
    int t = (int)(tiles * blockIdx.x / gridDim.x);
    int left = (int)(tiles * (blockIdx.x + 1) / gridDim.x) - t;
    for (int steps = (left + kRT - 1) / kRT; steps > 0; --steps) {
        const int n = (left + steps - 1) / steps;
        switch (n) {
        case 1: rows_block<1>(X, 16 * t, net, Y, lds); break;
        case 2: rows_block<2>(X, 16 * t, net, Y, lds); break;
        case 3: rows_block<3>(X, 16 * t, net, Y, lds); break;
        default: rows_block<kRT>(X, 16 * t, net, Y, lds); break;
        }
        t += n;
        left -= n;
    }
}

// Adam (Kingma & Ba 2015); c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t).
__global__ void k_adam(float *w, float *m, float *v, const float *g, int64_t n, float lr,
                       float beta1, float beta2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// Input-major copy of W (rows x cols, row-major): wt[c][r] = w[r][c].
__global__ void k_transpose(const float *w, int rows, int cols, float *wt)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)rows * cols) return;
    const int r = (int)(e / cols), c = (int)(e % cols);
    wt[(int64_t)c * rows + r] = w[e];
}

hipError_t launch_net_layout(const float *flat, float *net, hipStream_t s)
{
    // flat: W1 (256 x 1024), b1, W2 (256 x 256), b2, W3, b3
    // net:  W1, b1, W2^T (256 x 256), b2, W3, b3
    const int64_t n1 = (int64_t)kNetH * kNetIn, n2 = (int64_t)kNetH * kNetH;
    hipError_t e = hipMemcpyAsync(net, flat, sizeof(float) * (n1 + kNetH),
                                  hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_transpose, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, s,
                       flat + n1 + kNetH, kNetH, kNetH, net + n1 + kNetH);
    const int64_t tail = kNetParams - (n1 + kNetH + n2);
    return hipMemcpyAsync(net + n1 + kNetH + n2, flat + n1 + kNetH + n2, sizeof(float) * tail,
                          hipMemcpyDeviceToDevice, s);
}

}  // namespace asp

// ===========================================================================
// The trainer of the C ABI.
// ===========================================================================

using namespace asp;

struct asp_mlp {
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int bmax = 0, cus = 0;
    float *w = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;   // kNetParams each
    float *H1 = nullptr, *H2 = nullptr;
    float *dY = nullptr, *dH1 = nullptr, *dH2 = nullptr;
    double *loss = nullptr, *part = nullptr;                        // the sum; one per 16 rows
    int32_t *bad = nullptr;                                         // a row index out of range
    int64_t t = 0;                                                  // Adam steps taken
    std::string err;
};

namespace {

constexpr int64_t kOffB1 = (int64_t)kNetH * kNetIn;
constexpr int64_t kOffW2 = kOffB1 + kNetH;
constexpr int64_t kOffB2 = kOffW2 + (int64_t)kNetH * kNetH;
constexpr int64_t kOffW3 = kOffB2 + kNetH;
constexpr int64_t kOffB3 = kOffW3 + (int64_t)kNetOut * kNetH;
constexpr int64_t kRowsMax = (int64_t)1 << 24;   // rows of one forward launch
constexpr int64_t kRowsByLayer = 3072;
static_assert(kOffW2 % 4 == 0 && kOffW3 % 4 == 0, "16-byte rows of the weights");

asp_status mfail(asp_mlp *n, asp_status s, const std::string &msg)
{
    if (n) n->err = msg;
    return s;
}

#define MLP_HIP(n, call)                                                              \
    do {                                                                              \
        hipError_t e_ = (call);                                                       \
        if (e_ != hipSuccess)                                                         \
            return mfail((n), ASP_ERR_DEVICE, std::string(#call ": ") + hipGetErrorString(e_)); \
    } while (0)

// Rows picked by idx (or in order) of a caller's array of rows of `cols` floats.
Op rows_of(const float *p, int rows, int cols, const int32_t *idx, int64_t n_src, int32_t *bad)
{
    return Op{p, cols, rows, cols, idx, n_src, bad, ((uintptr_t)p & 15) == 0 ? 1 : 0};
}

Op weights(const float *w, int rows, int cols)
{
    return Op{w, cols, rows, cols, nullptr, 0, nullptr, 1};
}

// The two hidden layers of B rows into H1 and H2.
void hidden(asp_mlp *n, const Op &X)
{
    const float *w = n->w;
    const dim3 grid(kHTiles, (unsigned)((X.rows + kTile - 1) / kTile));
    hipLaunchKernelGGL(k_layer, grid, dim3(256), kGemmLds, n->stream, X, weights(w, kNetH, kNetIn),
                       w + kOffB1, n->H1);
    hipLaunchKernelGGL(k_layer, grid, dim3(256), kGemmLds, n->stream, weights(n->H1, X.rows, kNetH),
                       weights(w + kOffW2, kNetH, kNetH), w + kOffB2, n->H2);
}

// Loss (added to n->loss) and the full gradient into n->g for the B rows of x
// and t picked by idx (nullptr: the first B).
hipError_t forward_backward(asp_mlp *n, const float *x, const float *t, int64_t n_rows,
                            const int32_t *idx, int B)
{
    hipStream_t s = n->stream;
    const float *w = n->w;
    float *g = n->g;
    const Op X = rows_of(x, B, kNetIn, idx, n_rows, n->bad), T = rows_of(t, B, kNetOut, idx, n_rows, n->bad);
    const unsigned mt = (unsigned)((B + kTile - 1) / kTile), heads = (unsigned)((B + kHeadRows - 1) / kHeadRows);
    hidden(n, X);
    hipLaunchKernelGGL(k_head<true>, dim3(heads), dim3(256), 0, s, n->H2, w + kOffW3, w + kOffB3, T, n->dY,
                       n->dH2, n->part);
    const Back b{B, n->dY, n->H1, n->H2, w + kOffW2, n->dH2, n->dH1, g + kOffW2, g + kOffB2,
                 g + kOffW3, g + kOffB3};
    hipLaunchKernelGGL(k_back, dim3(kBackFixed + kHTiles * mt), dim3(256), kGemmLds, s, b);
    hipLaunchKernelGGL(k_back1, dim3(kHTiles * (kNetIn / kTile + 1) + 1), dim3(256), kGemmLds, s, X, n->dH1,
                       g, g + kOffB1, n->part, (int)heads, n->loss);
    return hipGetLastError();
}

// The forward pass layer by layer, at most bmax rows.  x has been read when y is
// written.
hipError_t forward_by_layer(asp_mlp *n, const float *x, int rows, float *y)
{
    const float *w = n->w;
    const Op X = rows_of(x, rows, kNetIn, nullptr, 0, nullptr);
    hidden(n, X);
    hipLaunchKernelGGL(k_head<false>, dim3((unsigned)((rows + kHeadRows - 1) / kHeadRows)), dim3(256), 0,
                       n->stream, n->H2, w + kOffW3, w + kOffB3, X, y, nullptr, nullptr);
    return hipGetLastError();
}

// The forward pass of all rows.  A few rows leave most CUs idle in k_rows, whose
// work-groups have all columns of a layer and take 54 us for up to 3072 rows;
// layer by layer the columns are spread too: 38 us for up to 1024 rows, 47 for
// 2048, 56 for 3072, 71 for 4096.  k_rows writes the outputs of some rows while
// it reads others, so outputs that lie within the inputs' memory (as a call may
// have them that keeps the rows in place) are formed layer by layer too, bmax
// rows at a time in order.
hipError_t forward(asp_mlp *n, const float *x, int64_t rows, float *y)
{
    if (rows == 0) return hipSuccess;      // a launch has no empty grid
    const float *w = n->w;
    if (rows <= n->bmax && rows <= kRowsByLayer) return forward_by_layer(n, x, (int)rows, y);
    const uintptr_t x0 = (uintptr_t)x, y0 = (uintptr_t)y;
    const bool apart = y0 + sizeof(float) * kNetOut * (uintptr_t)rows <= x0 ||
                       x0 + sizeof(float) * kNetIn * (uintptr_t)rows <= y0;
    if (!apart) {
        for (int64_t r = 0; r < rows; r += n->bmax) {
            const int M = (int)(rows - r < n->bmax ? rows - r : n->bmax);
            const hipError_t e = forward_by_layer(n, x + r * kNetIn, M, y + r * kNetOut);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const Net net{w, w + kOffB1, w + kOffW2, w + kOffB2, w + kOffW3, w + kOffB3};
    for (int64_t r = 0; r < rows; r += kRowsMax) {
        const int M = (int)(rows - r < kRowsMax ? rows - r : kRowsMax);
        const Op X = rows_of(x + r * kNetIn, M, kNetIn, nullptr, 0, nullptr);
        const int tiles = (M + 15) / 16;
        hipLaunchKernelGGL(k_rows, dim3((unsigned)(tiles < n->cus ? tiles : n->cus)), dim3(kRowThreads),
                           kRowsLds, n->stream, X, net, y + r * kNetOut);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t mlp_kernel_setup()
{
    const void *gemms[] = {(const void *)k_layer, (const void *)k_back, (const void *)k_back1};
    for (const void *k : gemms) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGemmLds);
        if (e != hipSuccess) return e;
    }
    return hipFuncSetAttribute((const void *)k_rows, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRowsLds);
}

void mlp_release(asp_mlp *n)
{
    if (!n) return;
    if (n->stream) (void)hipStreamSynchronize(n->stream);
    float *bufs[] = {n->w, n->g, n->m, n->v, n->H1, n->H2, n->dY, n->dH1, n->dH2};
    for (float *b : bufs) (void)hipFree(b);
    (void)hipFree(n->loss);
    (void)hipFree(n->part);
    (void)hipFree(n->bad);
    if (n->own_stream && n->stream) (void)hipStreamDestroy(n->stream);
}

}  // namespace

extern "C" {

asp_status asp_mlp_create(const float *init, int32_t max_batch, void *stream, asp_mlp **out)
{
    if (!out) return ASP_ERR_INVALID_ARG;
    *out = nullptr;
    if (!init || max_batch < 1 || max_batch > 65536) return ASP_ERR_INVALID_ARG;
    asp_mlp *n = new (std::nothrow) asp_mlp;
    if (!n) return ASP_ERR_NOMEM;
    n->bmax = max_batch;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n->cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        mlp_kernel_setup() != hipSuccess) {
        delete n;
        return ASP_ERR_DEVICE;
    }
    auto bail = [&](asp_status s) { mlp_release(n); delete n; return s; };
    if (stream) {
        n->stream = (hipStream_t)stream;
    } else {
        if (hipStreamCreate(&n->stream) != hipSuccess) return bail(ASP_ERR_DEVICE);
        n->own_stream = true;
    }
    const size_t P = sizeof(float) * kNetParams;
    const size_t B = (size_t)max_batch;
    if (hipMalloc(&n->w, P) != hipSuccess || hipMalloc(&n->g, P) != hipSuccess ||
        hipMalloc(&n->m, P) != hipSuccess || hipMalloc(&n->v, P) != hipSuccess ||
        hipMalloc(&n->H1, sizeof(float) * B * kNetH) != hipSuccess ||
        hipMalloc(&n->H2, sizeof(float) * B * kNetH) != hipSuccess ||
        hipMalloc(&n->dY, sizeof(float) * B * kNetOut) != hipSuccess ||
        hipMalloc(&n->dH1, sizeof(float) * B * kNetH) != hipSuccess ||
        hipMalloc(&n->dH2, sizeof(float) * B * kNetH) != hipSuccess ||
        hipMalloc(&n->loss, sizeof(double)) != hipSuccess ||
        hipMalloc(&n->part, sizeof(double) * ((B + kHeadRows - 1) / kHeadRows)) != hipSuccess ||
        hipMalloc(&n->bad, sizeof(int32_t)) != hipSuccess)
        return bail(ASP_ERR_NOMEM);
    if (hipMemcpyAsync(n->w, init, P, hipMemcpyHostToDevice, n->stream) != hipSuccess ||
        hipMemsetAsync(n->m, 0, P, n->stream) != hipSuccess ||
        hipMemsetAsync(n->v, 0, P, n->stream) != hipSuccess ||
        hipStreamSynchronize(n->stream) != hipSuccess)
        return bail(ASP_ERR_DEVICE);
    *out = n;
    return ASP_OK;
}

void asp_mlp_destroy(asp_mlp *n)
{
    mlp_release(n);
    delete n;
}

const char *asp_mlp_last_error(const asp_mlp *n)
{
    return n ? n->err.c_str() : "null network";
}

asp_status asp_mlp_weights(asp_mlp *n, float *out)
{
    if (!n || !out) return ASP_ERR_INVALID_ARG;
    MLP_HIP(n, hipMemcpyAsync(out, n->w, sizeof(float) * kNetParams, hipMemcpyDeviceToHost,
                              n->stream));
    MLP_HIP(n, hipStreamSynchronize(n->stream));
    return ASP_OK;
}

asp_status asp_mlp_loss_grad(asp_mlp *n, const float *x_dev, const float *t_dev, int32_t batch,
                             double *loss, float *grad)
{
    if (!n || !x_dev || !t_dev || batch < 1 || batch > n->bmax) return ASP_ERR_INVALID_ARG;
    MLP_HIP(n, hipMemsetAsync(n->loss, 0, sizeof(double), n->stream));
    MLP_HIP(n, forward_backward(n, x_dev, t_dev, batch, nullptr, batch));
    if (grad)
        MLP_HIP(n, hipMemcpyAsync(grad, n->g, sizeof(float) * kNetParams, hipMemcpyDeviceToHost,
                                  n->stream));
    double l = 0.0;
    MLP_HIP(n, hipMemcpyAsync(&l, n->loss, sizeof(double), hipMemcpyDeviceToHost, n->stream));
    MLP_HIP(n, hipStreamSynchronize(n->stream));
    if (loss) *loss = l;
    return ASP_OK;
}

asp_status asp_mlp_train(asp_mlp *n, const float *x_dev, const float *t_dev, int64_t n_rows,
                         const int32_t *order_dev, int64_t n_steps, int32_t batch, float lr,
                         double *mean_loss)
{
    if (!n || !x_dev || !t_dev || !order_dev || n_rows < 1 || n_steps < 0 || batch < 1 ||
        batch > n->bmax || !(lr > 0.0f))
        return ASP_ERR_INVALID_ARG;
    const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
    MLP_HIP(n, hipMemsetAsync(n->loss, 0, sizeof(double), n->stream));
    MLP_HIP(n, hipMemsetAsync(n->bad, 0, sizeof(int32_t), n->stream));
    for (int64_t st = 0; st < n_steps; ++st) {
        MLP_HIP(n, forward_backward(n, x_dev, t_dev, n_rows, order_dev + st * batch, batch));
        n->t += 1;
        const float c1 = (float)(1.0 / (1.0 - pow(0.9, (double)n->t)));
        const float c2 = (float)(1.0 / (1.0 - pow(0.999, (double)n->t)));
        hipLaunchKernelGGL(k_adam, dim3((unsigned)((kNetParams + 255) / 256)), dim3(256), 0,
                           n->stream, n->w, n->m, n->v, n->g, kNetParams, lr, beta1, beta2, eps,
                           c1, c2);
        MLP_HIP(n, hipGetLastError());
    }
    double l = 0.0;
    int32_t bad = 0;
    MLP_HIP(n, hipMemcpyAsync(&l, n->loss, sizeof(double), hipMemcpyDeviceToHost, n->stream));
    MLP_HIP(n, hipMemcpyAsync(&bad, n->bad, sizeof(int32_t), hipMemcpyDeviceToHost, n->stream));
    MLP_HIP(n, hipStreamSynchronize(n->stream));
    if (mean_loss) *mean_loss = n_steps > 0 ? l / (double)n_steps : 0.0;
    if (bad) return mfail(n, ASP_ERR_INVALID_ARG, "a sample index lies outside the data");
    return ASP_OK;
}

asp_status asp_mlp_forward(asp_mlp *n, const float *x_dev, int64_t rows, float *y_dev)
{
    if (!n || (!x_dev && rows > 0) || (!y_dev && rows > 0) || rows < 0) return ASP_ERR_INVALID_ARG;
    MLP_HIP(n, forward(n, x_dev, rows, y_dev));
    MLP_HIP(n, hipStreamSynchronize(n->stream));
    return ASP_OK;
}

}  // extern "C"
