// Learned screen: an MLP that predicts log|psi(x')| of a connected
// configuration from the occupation bits of x' and one-hot codes of its
// excitation indices, trained on amplitudes the network itself produces, so
// that connections predicted far below the sample's own amplitude can skip
// the transformer.  (The paper's only filter is the sample-aware restriction
// of Section 3.4 item 4; this is an addition.)
//
//   u  = [bits(x') | onehot(i) | onehot(j) | onehot(a) | onehot(b)]   (5N)
//   z1 = GELU(u W1 + b1), z2 = GELU(z1 W2 + b2), y = z2 . w3 + b3
//
// Master weights and Adam moments are FP64 on the device.  Forward and
// gradient run in FP64 (parity path) or FP32; every reduction has a fixed
// order, so results are reproducible.  The inference kernel used inside the
// full local energy computes the first layer in FP32 from the sparse input
// and the hidden layer with BF16 MFMA, FP32 accumulation.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "internal.hpp"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct nnqs_screen {
    int N = 0, H = 0;
    int64_t count = 0;
    double *w = nullptr, *m = nullptr, *v = nullptr;  // FP64 master weights and Adam moments
    int64_t t = 0;                                     // Adam step count
    float *w32 = nullptr;                              // FP32 copy (W1 b1 b2 w3 b3 read by inference)
    __bf16 *w2t = nullptr;                             // BF16 W2 transposed [H][H] (n-major)
    float *cw1 = nullptr;                              // combined first-layer rows [4][N][H] (inference)
    uint8_t *w2f8 = nullptr;                           // FP8 E4M3 W2 transposed [H][H], scaled
    float *w2scale = nullptr;                          // {2^k applied to W2, 2^-k applied to products}
    float *gelu_tab = nullptr;                         // GELU table (512 pairs) of the inference kernel
    bool infer_dirty = true;
    // scratch (grown on demand): activations for gradients
    void *scratch = nullptr;
    size_t scratch_bytes = 0;
    // scratch of the fallback judge (predictions and reduction partials)
    void *jscratch = nullptr;
    size_t jscratch_bytes = 0;
};

namespace nnqs {

struct ScreenOff {
    int64_t W1, b1, W2, b2, w3, b3, total;
};

__host__ __device__ inline ScreenOff screen_off(int N, int H) {
    ScreenOff o{};
    o.W1 = 0;
    o.b1 = (int64_t)5 * N * H;
    o.W2 = o.b1 + H;
    o.b2 = o.W2 + (int64_t)H * H;
    o.w3 = o.b2 + H;
    o.b3 = o.w3 + H;
    o.total = o.b3 + 1;
    return o;
}

template <typename T> __device__ __forceinline__ T gelu_t(T v);
template <> __device__ __forceinline__ double gelu_t<double>(double v) {
    return 0.5 * v * (1.0 + erf(v * 0.70710678118654752440));
}
template <> __device__ __forceinline__ float gelu_t<float>(float v) {
    return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
}
template <typename T> __device__ __forceinline__ T gelu_grad_t(T v) {
    const T cdf = T(0.5) * (T(1) + (sizeof(T) == 8 ? (T)erf((double)v * 0.70710678118654752440)
                                                    : (T)erff((float)v * 0.70710678118654752f)));
    const T pdf = (sizeof(T) == 8 ? (T)exp(-0.5 * (double)v * (double)v) : (T)__expf(-0.5f * (float)v * (float)v)) *
                  T(0.39894228040143267794);
    return cdf + v * pdf;
}

// Active inputs of example k: the set bits of x' and up to four one-hot codes.
struct ScreenInput {
    Key x;
    uint8_t e[4];
};

__device__ __forceinline__ ScreenInput load_input(const uint64_t *keys, const uint8_t *exc, int64_t k) {
    ScreenInput in;
    in.x.lo = keys[2 * k];
    in.x.hi = keys[2 * k + 1];
    for (int t = 0; t < 4; t++) in.e[t] = exc[4 * k + t];
    return in;
}

// ------------------------------------------------- forward and gradient
// The training path: dense products on the 16x16x4 matrix instruction of the
// precision (FP64, or FP32, whose result is the chain of fused multiply-adds
// in ascending k, checked against fmaf over normal and denormal values).  A
// minibatch step is six launches: the FP32 weights, layer 1 from the sparse
// input, the hidden product, the output with its gradient, the hidden
// product's transpose, and every weight and bias gradient together.  With
// one output element per thread, a launch per elementwise pass and four-block
// column sums a step of 4,096 pairs at N = 120, hidden 256 took 950 us; now
// 164 us, the choice of the minibatch included.
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mma;
template <> struct Mma<float> {
    typedef f32x4 Acc;
    static __device__ __forceinline__ Acc mul(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lk, int i) { return 4 * lk + i; }  // row of accumulator i
};
template <> struct Mma<double> {
    typedef f64x4 Acc;
    static __device__ __forceinline__ Acc mul(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lk, int i) { return lk + 4 * i; }
};

__global__ void k_convert_f32(const double *__restrict__ s, float *__restrict__ d, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) d[k] = (float)s[k];
}

// a1[k][c] = b1[c] + sum over active inputs p of W1[p][c] in ascending p, and
// z1 = GELU(a1).  One wave per example (its inputs are then the same for all
// lanes, and the rows of eight of them load together), 256 columns per pass;
// 44 rows of 1 KB from L2 bound it.  30 us with a thread per element and one
// dependent load at a time, now 13 us (4,096 examples, N = 120).
template <typename T>
__global__ void __launch_bounds__(256) k_screen_layer1(int N, int H, const T *__restrict__ w,
                                                       const uint64_t *__restrict__ keys,
                                                       const uint8_t *__restrict__ exc, int64_t n,
                                                       T *__restrict__ a1, T *__restrict__ z1) {
    const int lane = threadIdx.x & 63;
    const int64_t k = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (k >= n) return;
    const ScreenOff o = screen_off(N, H);
    const ScreenInput in = load_input(keys, exc, k);
    const uint64_t lo_in = N >= 64 ? in.x.lo : in.x.lo & ((1ull << N) - 1);
    const uint64_t hi_in = N >= 128 ? in.x.hi : N > 64 ? in.x.hi & ((1ull << (N - 64)) - 1) : 0ull;
    for (int c0 = 0; c0 < H; c0 += 256) {
        int c[4];
        T acc[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            c[j] = std::min(c0 + lane + 64 * j, H - 1);
            acc[j] = w[o.b1 + c[j]];
        }
        uint64_t lo = lo_in, hi = hi_in;
        while (lo | hi) {
            int p[8];
            T v[8][4];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                p[u] = -1;
                if (lo) {
                    p[u] = __ffsll((unsigned long long)lo) - 1;
                    lo &= lo - 1;
                } else if (hi) {
                    p[u] = 63 + __ffsll((unsigned long long)hi);
                    hi &= hi - 1;
                }
#pragma unroll
                for (int j = 0; j < 4; j++) v[u][j] = w[o.W1 + (int64_t)std::max(p[u], 0) * H + c[j]];
            }
            __builtin_amdgcn_sched_barrier(0);  // all loads before the first sum
#pragma unroll
            for (int u = 0; u < 8; u++)
#pragma unroll
                for (int j = 0; j < 4; j++) acc[j] = p[u] >= 0 ? acc[j] + v[u][j] : acc[j];
        }
#pragma unroll
        for (int t = 0; t < 4; t++)  // 255 (absent) and any other code >= N add nothing
            if (in.e[t] < N)
#pragma unroll
                for (int j = 0; j < 4; j++) acc[j] += w[o.W1 + (int64_t)((t + 1) * N + in.e[t]) * H + c[j]];
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (c0 + lane + 64 * j < H) {
                if (a1) a1[k * H + c[j]] = acc[j];
                z1[k * H + c[j]] = gelu_t<T>(acc[j]);
            }
    }
}

// The hidden layer's product and its transpose, 32 x 64 per block, each wave
// 16 x 32: with W, a2 = A W2 + b2 (kept if asked for) and out = GELU(a2); with
// kBack, out = (A W2^T) GELU'(act).  Depth in slices of 64 through LDS, the
// next slice's loads in flight (rows padded to 68 and 81: the fragments, and
// the transposed store, then touch every bank once).  4,096 x 256 x 256 in
// FP32: 85 us with one element per thread, now 15 us (512 blocks, four slices
// of one memory latency each; the matrix instructions take 3.4 us of it).
// The blocks past the row tiles of kBack's launch form the partial sums of the
// output weights' gradient over all `total` rows (z2 and gy begin at the first),
// w3p[ph][c] = sum of gy[k] z2[k][c] over k = ph, ph + 16, ...: 64 columns of
// one phase each, one wave (a CU takes in few lines at a time, so the sums want
// many CUs more than full ones).
template <typename T, bool kBack>
__global__ void __launch_bounds__(256) k_screen_hidden(const T *__restrict__ A, const T *__restrict__ W,
                                                       const T *__restrict__ bias, const T *__restrict__ act, int64_t n,
                                                       int H, T *__restrict__ a2, T *__restrict__ out,
                                                       const T *__restrict__ z2, const T *__restrict__ gy, int64_t total,
                                                       double *__restrict__ w3p) {
    __shared__ T As[32][68];
    __shared__ T Ws[64][81];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lr = l & 15, lk = l >> 4, rw = 16 * (w & 1), cw = 32 * (w >> 1);
    const int64_t r0 = (int64_t)blockIdx.x * 32;
    const int c0 = blockIdx.y * 64;
    if (kBack && r0 >= n) {
        const int ph = (int)((int64_t)blockIdx.x - (n + 31) / 32), c = std::min(c0 + l, H - 1);
        if (w > 0) return;
        double s = 0.0;
        constexpr int kU = 32;  // loads in flight
        for (int64_t k0 = ph; k0 < total; k0 += 16 * kU) {
            T v[kU], g[kU];
#pragma unroll
            for (int u = 0; u < kU; u++) {
                const int64_t k = std::min(k0 + 16 * u, total - 1);
                v[u] = z2[k * H + c];
                g[u] = gy[k];
            }
            __builtin_amdgcn_sched_barrier(0);  // the compiler would wait for each load before the next
#pragma unroll
            for (int u = 0; u < kU; u++)
                if (k0 + 16 * u < total) s += (double)(v[u] * g[u]);
        }
        if (c0 + l < H) w3p[ph * H + c0 + l] = s;
        return;
    }
    T pa[8], pw[16];
    auto load = [&](int k0) {
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int64_t r = r0 + w + 4 * e;
            pa[e] = r < n && k0 + l < H ? A[r * H + k0 + l] : T(0);
        }
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int c = c0 + (kBack ? w + 4 * e : l), k = k0 + (kBack ? l : w + 4 * e);
            pw[e] = c < H && k < H ? W[kBack ? (int64_t)c * H + k : (int64_t)k * H + c] : T(0);
        }
    };
    typename Mma<T>::Acc acc[2] = {};
    load(0);
    for (int k0 = 0; k0 < H; k0 += 64) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; e++) As[w + 4 * e][l] = pa[e];
#pragma unroll
        for (int e = 0; e < 16; e++) {
            if (kBack) Ws[l][w + 4 * e] = pw[e];
            else Ws[w + 4 * e][l] = pw[e];
        }
        __syncthreads();
        if (k0 + 64 < H) load(k0 + 64);
        T a[16], b[16][2];
#pragma unroll
        for (int q = 0; q < 16; q++) {
            a[q] = As[rw + lr][4 * q + lk];
            b[q][0] = Ws[4 * q + lk][cw + lr];
            b[q][1] = Ws[4 * q + lk][cw + 16 + lr];
        }
        __builtin_amdgcn_sched_barrier(0);  // one LDS latency, not sixteen
#pragma unroll
        for (int q = 0; q < 16; q++)
#pragma unroll
            for (int cb = 0; cb < 2; cb++) acc[cb] = Mma<T>::mul(a[q], b[q][cb], acc[cb]);
    }
#pragma unroll
    for (int cb = 0; cb < 2; cb++) {
        const int c = c0 + cw + cb * 16 + lr;
        if (c >= H) continue;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t r = r0 + rw + Mma<T>::row(lk, i);
            if (r >= n) continue;
            if (kBack) {
                out[r * H + c] = acc[cb][i] * gelu_grad_t<T>(act[r * H + c]);
            } else {
                const T v = acc[cb][i] + bias[c];
                if (a2) a2[r * H + c] = v;
                out[r * H + c] = gelu_t<T>(v);
            }
        }
    }
}

// y[k] = b3 + sum_c z2[k][c] w3[c] in ascending c; with `target`, gy[k] = 2
// (y_k - target_k) / total and d2[k][c] = gy[k] w3[c] GELU'(a2[k][c]).  Sixteen
// examples per block: their rows go through LDS, where 16 lanes follow one
// chain each (the chain bounds it: 57 us when every lane also made its 256
// GELUs in the chain, now 9 us).
template <typename T>
__global__ void __launch_bounds__(256) k_screen_out(const T *__restrict__ a2, const T *__restrict__ z2,
                                                    const T *__restrict__ w, int N, int H, int64_t n, int64_t total,
                                                    const double *__restrict__ target, T *__restrict__ y,
                                                    double *__restrict__ pred, T *__restrict__ gy,
                                                    T *__restrict__ d2) {
    __shared__ T zs[16][257];
    __shared__ T ws[256];
    __shared__ T gs[16];
    const ScreenOff o = screen_off(N, H);
    const int64_t k0 = (int64_t)blockIdx.x * 16;
    const int t = threadIdx.x;
    const int rows = (int)std::min<int64_t>(16, n - k0);
    T av[16];  // a2 of column c
    auto load_a2 = [&](int c) {
#pragma unroll
        for (int r = 0; r < 16; r++) av[r] = c < H ? a2[(k0 + std::min(r, rows - 1)) * H + c] : T(0);
    };
    if (target) load_a2(t);  // in flight while the chain runs
    T acc = w[o.b3];
    for (int c0 = 0; c0 < H; c0 += 256) {
        const int c = c0 + t, cnt = std::min(256, H - c0);
        __syncthreads();
        T zv[16];
#pragma unroll
        for (int r = 0; r < 16; r++) zv[r] = c < H ? z2[(k0 + std::min(r, rows - 1)) * H + c] : T(0);
        ws[t] = c < H ? w[o.w3 + c] : T(0);
        __builtin_amdgcn_sched_barrier(0);  // all loads before the first store
#pragma unroll
        for (int r = 0; r < 16; r++) zs[r][t] = zv[r];
        __syncthreads();
        if (t < 16) {
#pragma unroll 16
            for (int q = 0; q < cnt; q++) acc += zs[t][q] * ws[q];
        }
    }
    if (t < 16 && k0 + t < n) {
        y[k0 + t] = acc;
        if (pred) pred[k0 + t] = (double)acc;
        if (target) {
            const T g = (T)(2.0 * ((double)acc - target[k0 + t]) / (double)total);
            gy[k0 + t] = g;
            gs[t] = g;
        }
    }
    if (!target) return;
    __syncthreads();
    for (int c = t; c < H; c += 256) {
        if (c != t) load_a2(c);
        const T w3 = w[o.w3 + c];
#pragma unroll
        for (int r = 0; r < 16; r++)
            if (r < rows) d2[(k0 + r) * H + c] = gs[r] * w3 * gelu_grad_t<T>(av[r]);
    }
}

// One 32 x 32 tile of gW1 = X^T d1 (kFirst) or gW2 = z1^T d2, 16 x 16 a wave:
// a chain of matrix instructions over the n examples (ascending, as a plain sum
// would).  Slices of 64 examples go through LDS, the loads of three in flight.
// X is the input as a dense 0/1 matrix (bits of x', then the one-hot fields of
// i, j, a, b), formed from one byte of the example per element.  The tiles of
// the first row also add up D's columns, for the biases: 16 row phases per
// column, combined in phase order.
constexpr int kSlice = 64, kAhead = 3;
template <typename T> struct TileLds {  // rows padded to 48: the fragments touch every bank once
    T A[2][kSlice][48], D[2][kSlice][48];
};

template <typename T, bool kFirst>
__device__ __forceinline__ void screen_tile(TileLds<T> &lds, int N, int H, const uint64_t *__restrict__ keys,
                                            const uint8_t *__restrict__ exc, int64_t n, const T *__restrict__ z1,
                                            const T *__restrict__ D, int i0, int j0, double *__restrict__ out,
                                            double *__restrict__ colsum) {
    auto &As = lds.A, &Ds = lds.D;
    typedef typename std::conditional<kFirst, uint8_t, T>::type S;
    const int t = threadIdx.x, l = t & 63, w = t >> 6, lr = l & 15, lk = l >> 4;
    const int M = kFirst ? 5 * N : H;
    // element (k, column t & 31) of a slice: k = (t >> 5) + 8 e; columns beyond the matrix repeat its last
    const int rk = t >> 5, p = std::min(i0 + (t & 31), M - 1);
    const int dc = std::min(t & 31, H - 1 - j0), field = p / N, bit = p - field * N;
    const S *A;
    int as;  // elements per example
    if constexpr (kFirst) {
        A = field == 0 ? reinterpret_cast<const uint8_t *>(keys) + (bit >> 3) : exc + field - 1;
        as = field == 0 ? 16 : 4;
    } else {
        A = z1 + p;
        as = H;
    }
    D += j0;
    // A slice's loads share a row pointer and fixed lane offsets.  The last
    // slice's offsets hold to the last example and the slices past it repeat
    // it; rows beyond n become zero on the way to LDS.
    uint32_t ao[8], od[8];
    auto offsets = [&](int last) {
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int k = std::min(rk + 8 * e, last);
            ao[e] = (uint32_t)(k * as);
            od[e] = (uint32_t)(k * H + dc);
        }
    };
    offsets(kSlice);
    const int64_t slices = (n + kSlice - 1) / kSlice, klast = (slices - 1) * kSlice;
    S pa[kAhead][8];
    T pd[kAhead][8];
    auto load = [&](int q, int64_t k0) {
        if (k0 == klast) offsets((int)(n - 1 - klast));
        const int64_t kb = std::min(k0, klast);
        const S *Ak = A + kb * as;
        const T *Dk = D + kb * H;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            pa[q][e] = Ak[ao[e]];
            pd[q][e] = Dk[od[e]];
        }
    };
    double cs[2] = {0.0, 0.0};  // row phases rk and rk + 8
    auto store = [&](int q, int slot, int64_t k0) {
        const int rem = (int)std::min<int64_t>(n - k0, kSlice) - rk;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            T av;
            if constexpr (kFirst)
                av = (field == 0 ? (pa[q][e] >> (bit & 7)) & 1 : pa[q][e] == bit) ? T(1) : T(0);
            else
                av = pa[q][e];
            const T dv = 8 * e < rem ? pd[q][e] : T(0);
            As[slot][rk + 8 * e][t & 31] = 8 * e < rem ? av : T(0);
            Ds[slot][rk + 8 * e][t & 31] = dv;
            cs[e & 1] += (double)dv;
        }
    };
    typename Mma<T>::Acc acc = {};
    const int rw = 16 * (w & 1), cw = 16 * (w >> 1);
#pragma unroll
    for (int q = 0; q < kAhead; q++) load(q, q * kSlice);
    store(0, 0, 0);
    for (int64_t s0 = 0; s0 < slices; s0 += 2 * kAhead)
#pragma unroll
        for (int u = 0; u < 2 * kAhead; u++) {  // slice s0 + u (zeros past the last) is in slot u & 1, the next
                                                // in registers (u + 1) % kAhead
            __syncthreads();  // the slice is written, the other slot read
            T a[kSlice / 4], d[kSlice / 4];
#pragma unroll
            for (int q = 0; q < kSlice / 4; q++) {
                a[q] = As[u & 1][4 * q + lk][rw + lr];
                d[q] = Ds[u & 1][4 * q + lk][cw + lr];
            }
            load(u % kAhead, (s0 + u + kAhead) * kSlice);
            __builtin_amdgcn_sched_barrier(0);  // reads and loads stay ahead of the products
            store((u + 1) % kAhead, (u + 1) & 1, (s0 + u + 1) * kSlice);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < kSlice / 4; q++) acc = Mma<T>::mul(a[q], d[q], acc);
        }
    const int j = j0 + cw + lr;
    if (j < H)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int r = i0 + rw + Mma<T>::row(lk, i);
            if (r < M) out[(int64_t)r * H + j] = (double)acc[i];
        }
    if (i0 == 0) {
        double(*part)[32] = reinterpret_cast<double(*)[32]>(As);  // 16 phases
        __syncthreads();
        part[rk][t & 31] = cs[0];
        part[rk + 8][t & 31] = cs[1];
        __syncthreads();
        if (t < 32 && j0 + t < H) {
            double s = 0.0;
            for (int q = 0; q < 16; q++) s += part[q][t];
            colsum[j0 + t] = s;
        }
    }
}

// Every gradient of the weights and biases in one launch, so that its few
// tiles per matrix fill the chip together.  Blocks in order: b3 (the sum of
// gy) and w3 (its partial sums in phase order); the loss; the tiles of gW1 and
// gW2 with b1 and b2.  n / 4 matrix instructions of 32 cycles in a row bound
// it, 14 us for 4,096 examples.  The two products took 300 us, the sums 250 us,
// now 59 us together (with X in memory and the column sums in blocks of
// their own 96 us: a CU waits for about 21 ns per line there).
template <typename T>
__global__ void __launch_bounds__(256) k_screen_grads(int N, int H, const uint64_t *__restrict__ keys,
                                                      const uint8_t *__restrict__ exc,
                                                      const double *__restrict__ target, int64_t n,
                                                      const T *__restrict__ z1, const T *__restrict__ d1,
                                                      const T *__restrict__ d2, const T *__restrict__ y,
                                                      const T *__restrict__ gy, const double *__restrict__ w3p,
                                                      double *__restrict__ grad, double *__restrict__ loss) {
    __shared__ TileLds<T> lds;
    double *part = reinterpret_cast<double *>(&lds);
    const ScreenOff o = screen_off(N, H);
    const int t = threadIdx.x;
    int b = (int)blockIdx.x;
    if (b == 0) {  // strided partials, then a fixed-order tree
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        for (int64_t k = t; k < n; k += 4096) {
            T v[16];
#pragma unroll
            for (int q = 0; q < 16; q++) v[q] = gy[std::min(k + 256 * q, n - 1)];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 16; q++)
                if (k + 256 * q < n) s[q & 3] += (double)v[q];
        }
#pragma unroll
        for (int q = 0; q < 4; q++) part[t + 256 * q] = s[q];
        __syncthreads();
        for (int w = 512; w >= 1; w >>= 1) {
            for (int q = t; q < w; q += 256) part[q] += part[q + w];
            __syncthreads();
        }
        if (t == 0) grad[o.b3] = part[0];
        for (int c = t; c < H; c += 256) {
            double v = 0.0;
#pragma unroll
            for (int ph = 0; ph < 16; ph++) v += w3p[ph * H + c];
            grad[o.w3 + c] = v;
        }
        return;
    }
    if (b == 1) {
        if (!loss) return;
        double s = 0.0;
#pragma unroll 8
        for (int64_t k = t; k < n; k += 256) {
            const double r = (double)y[k] - target[k];
            s += r * r;
        }
        part[t] = s;
        __syncthreads();
        for (int w = 128; w >= 1; w >>= 1) {
            if (t < w) part[t] += part[t + w];
            __syncthreads();
        }
        if (t == 0) *loss = part[0] / (double)n;
        return;
    }
    b -= 2;
    const int jt = (H + 31) / 32, tiles1 = (5 * N + 31) / 32 * jt;
    if (b < tiles1)
        screen_tile<T, true>(lds, N, H, keys, exc, n, z1, d1, b / jt * 32, b % jt * 32, grad + o.W1, grad + o.b1);
    else
        screen_tile<T, false>(lds, N, H, keys, exc, n, z1, d2, (b - tiles1) / jt * 32, (b - tiles1) % jt * 32, grad + o.W2,
                              grad + o.b2);
}

template <typename T>
__global__ void k_to_double(const T *__restrict__ s, double *__restrict__ d, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) d[k] = (double)s[k];
}

__global__ void k_adam(double *__restrict__ w, const double *__restrict__ g, double *__restrict__ m,
                       double *__restrict__ v, int64_t n, double lr, double b1, double b2, double eps, double c1,
                       double c2) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    m[q] = b1 * m[q] + (1.0 - b1) * g[q];
    v[q] = b2 * v[q] + (1.0 - b2) * g[q] * g[q];
    w[q] -= lr * (m[q] / c1) / (sqrt(v[q] / c2) + eps);
}

__global__ void k_refresh_infer(const double *__restrict__ w, int N, int H, float *__restrict__ w32,
                                __bf16 *__restrict__ w2t) {
    const ScreenOff o = screen_off(N, H);
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < o.total) w32[e] = (float)w[e];
    if (e < (int64_t)H * H) {
        const int nn = (int)(e / H), k = (int)(e % H);
        w2t[e] = (__bf16)(float)w[o.W2 + (int64_t)k * H + nn];  // w2t[n][k] = W2[k][n]
    }
}

// --------------------------------------------------------------- inference
// 16 connections per wave: first layer from the sparse input in FP32, into
// LDS as BF16; hidden layer with v_mfma_f32_16x16x32_bf16 (B tiles from the
// transposed BF16 W2 in L2); output dot product by DPP row sums.
constexpr int kScreenH = 256;

__device__ __forceinline__ float dpp_sum16(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));
    return v;
}

// GELU of the inference kernel, v * Phi(v), with the normal CDF Phi from a
// 512-entry table of (value, step) pairs on [-8, 8) and linear
// interpolation (error <= 3e-5, far below the BF16 / FP8 rounding of the
// result); the table lives in LDS.
constexpr int kSGeluN = 512;
constexpr float kSGeluScale = 32.0f, kSGeluOff = 256.0f, kSGeluMaxU = 511.99997f;

__device__ __forceinline__ float sgelu(const float2 *tab, float v) {
    const float u = __builtin_amdgcn_fmed3f(fmaf(v, kSGeluScale, kSGeluOff), 0.0f, kSGeluMaxU);
    const float2 e = tab[(int)u];
    return v * fmaf(__builtin_amdgcn_fractf(u), e.y, e.x);
}

// Lane 0's value of a 64-bit word, for every lane.
__device__ __forceinline__ uint64_t lane0_u64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 0);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 0);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t fp8x4(float a, float b, float c, float d) {  // OCP E4M3, saturated
    a = __builtin_amdgcn_fmed3f(a, -448.f, 448.f);
    b = __builtin_amdgcn_fmed3f(b, -448.f, 448.f);
    c = __builtin_amdgcn_fmed3f(c, -448.f, 448.f);
    d = __builtin_amdgcn_fmed3f(d, -448.f, 448.f);
    int v = 0;
    v = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, v, false);
    v = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, v, true);
    return (uint32_t)v;
}

// Inference: each wave takes one contiguous run of connections, 16 at a
// time.  The connections of one sample x are contiguous and x' differs from
// x only in the excitation's bits, so the first layer is
//   b1 + sum_{p in x} W1[p]   (per run sample, kept in LDS)
//   + sum_t C_t[e_t],  C_t = W1[one-hot block t + 1] + s_t W1[bit block],
// s_t = -1 for the annihilated i, j and +1 for the created a, b: four
// precombined rows per connection.  Lane l computes, for connection l & 15 of
// a group of 16, the units 32 ks + 8 (l >> 4) + j (ks < 8, j < 8): exactly the
// A operand of the hidden layer's v_mfma_f32_16x16x32_bf16 (or _fp8_fp8), so
// the GELU outputs stay in registers.  W2 (transposed, BF16 or FP8 with a
// per-tensor power-of-two scale) is loaded into LDS once per block and every
// B fragment is read from there; the output dot product by DPP row sums.
constexpr int kScreenWaves = 12;  // waves per block (one block per CU, three waves per SIMD)

template <bool kFp8>
__global__ void __launch_bounds__(64 * kScreenWaves) k_screen_infer(int N, const float *__restrict__ w32,
                                                                    const float *__restrict__ cw1,
                                                                    const __bf16 *__restrict__ w2t,
                                                                    const uint8_t *__restrict__ w2f8,
                                                                    const float *__restrict__ w2inv,
                                                                    const float *__restrict__ gelu_tab,
                                                                    const uint64_t *__restrict__ keys,
                                                                    const uint8_t *__restrict__ exc, int64_t n,
                                                                    float *__restrict__ pred) {
    constexpr int H = kScreenH;
    constexpr int WLD = kFp8 ? H + 16 : H + 8;  // LDS row length (elements) of W2^T, 16 bytes of padding
    typedef typename std::conditional<kFp8, uint8_t, __bf16>::type WT;
    typedef typename std::conditional<kFp8, long, bf16x8>::type AF;  // one A / B fragment per lane
    __shared__ __align__(16) WT w2s[H * WLD];
    __shared__ __align__(16) float basev[kScreenWaves][H];  // per wave: b1 + W1 rows of the run's sample
    __shared__ __align__(16) float2 gtab[kSGeluN];
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c16 = l & 15, q = l >> 4, r0 = 4 * q, kq = 8 * q;
    for (int i = threadIdx.x; i < kSGeluN; i += blockDim.x) gtab[i] = make_float2(gelu_tab[2 * i], gelu_tab[2 * i + 1]);
    {  // W2^T rows (output unit, k) into LDS, 16 bytes per load
        constexpr int per_row = H * (int)sizeof(WT) / 16;
        const uint8_t *src = kFp8 ? w2f8 : reinterpret_cast<const uint8_t *>(w2t);
        for (int i = threadIdx.x; i < H * per_row; i += blockDim.x) {
            const int r = i / per_row, c = i - r * per_row;
            *reinterpret_cast<uint4 *>(reinterpret_cast<uint8_t *>(w2s + r * WLD) + 16 * c) =
                *reinterpret_cast<const uint4 *>(src + (int64_t)r * H * sizeof(WT) + 16 * c);
        }
    }
    __syncthreads();
    float *bv = basev[w];
    const ScreenOff o = screen_off(N, H);
    const float inv2 = kFp8 ? w2inv[0] : 1.0f;
    const int64_t nwaves = (int64_t)gridDim.x * kScreenWaves, wid = (int64_t)blockIdx.x * kScreenWaves + w;
    const int64_t per = (((n + nwaves - 1) / nwaves) + 15) & ~(int64_t)15;
    const int64_t beg = wid * per, end = beg + per < n ? beg + per : n;
    Key ref;
    ref.lo = ref.hi = 0ull;
    bool have_ref = false;
    // this lane's units: 32 ks + kq + j
    auto add_row = [&](float(&acc)[8][8], const float *row) {
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            const float4 lo = *reinterpret_cast<const float4 *>(row + 32 * ks + kq);
            const float4 hi = *reinterpret_cast<const float4 *>(row + 32 * ks + kq + 4);
            acc[ks][0] += lo.x;
            acc[ks][1] += lo.y;
            acc[ks][2] += lo.z;
            acc[ks][3] += lo.w;
            acc[ks][4] += hi.x;
            acc[ks][5] += hi.y;
            acc[ks][6] += hi.z;
            acc[ks][7] += hi.w;
        }
    };
    for (int64_t base = beg; base < end; base += 16) {
        // layer 1 for connection k = base + c16
        const int64_t k = base + c16;
        const bool ok = k < end;
        Key x;
        x.lo = ok ? keys[2 * k] : 0ull;
        x.hi = ok ? keys[2 * k + 1] : 0ull;
        uint8_t e4[4] = {255, 255, 255, 255};
        if (ok)
            for (int t = 0; t < 4; t++) e4[t] = exc[4 * k + t];
        // flipped bits (codes below N) and the sample x0 = x' ^ flips
        Key fm;
        fm.lo = fm.hi = 0ull;
        for (int t = 0; t < 4; t++)
            if (e4[t] < N) key_flip(fm, e4[t]);
        Key x0;
        x0.lo = x.lo ^ fm.lo;
        x0.hi = x.hi ^ fm.hi;
        // the run's reference sample is that of the group's first row (lane 0)
        // (the readlane builtin moves 32 bits: each word goes in two halves)
        const uint64_t rlo = lane0_u64(x0.lo), rhi = lane0_u64(x0.hi);
        if (!have_ref || rlo != ref.lo || rhi != ref.hi) {
            ref.lo = rlo;
            ref.hi = rhi;
            have_ref = true;
            float s4[4];
#pragma unroll
            for (int u = 0; u < 4; u++) s4[u] = w32[o.b1 + 4 * l + u];
            for (int wd = 0; wd < 2; wd++) {
                uint64_t m = wd ? ref.hi : ref.lo;
                while (m) {
                    const int bt = __ffsll((unsigned long long)m) - 1;
                    m &= m - 1;
                    const int p = wd * 64 + bt;
                    if (p >= N) break;  // bits above the spin orbitals carry no input
                    const float *row = w32 + o.W1 + (int64_t)p * H + 4 * l;
#pragma unroll
                    for (int u = 0; u < 4; u++) s4[u] += row[u];
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();  // earlier readers of bv are done
#pragma unroll
            for (int u = 0; u < 4; u++) bv[4 * l + u] = s4[u];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        float acc[8][8];
        if (x0.lo == ref.lo && x0.hi == ref.hi) {
#pragma unroll
            for (int ks = 0; ks < 8; ks++)
#pragma unroll
                for (int j = 0; j < 8; j++) acc[ks][j] = bv[32 * ks + kq + j];
#pragma unroll 1
            for (int t = 0; t < 4; t++)
                if (e4[t] < N) add_row(acc, cw1 + ((int64_t)t * N + e4[t]) * H);
        } else {  // another sample inside the group: the plain sum over the bits of x' and the one-hots
#pragma unroll
            for (int ks = 0; ks < 8; ks++)
#pragma unroll
                for (int j = 0; j < 8; j++) acc[ks][j] = w32[o.b1 + 32 * ks + kq + j];
            for (int wd = 0; wd < 2; wd++) {
                uint64_t m = wd ? x.hi : x.lo;
                while (m) {
                    const int bt = __ffsll((unsigned long long)m) - 1;
                    m &= m - 1;
                    const int p = wd * 64 + bt;
                    if (p >= N) break;
                    add_row(acc, w32 + o.W1 + (int64_t)p * H);
                }
            }
#pragma unroll 1
            for (int t = 0; t < 4; t++)
                if (e4[t] < N) add_row(acc, w32 + o.W1 + (int64_t)((t + 1) * N + e4[t]) * H);
        }
        AF af[8];
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            if constexpr (kFp8) {
                const uint32_t lo = fp8x4(sgelu(gtab, acc[ks][0]), sgelu(gtab, acc[ks][1]), sgelu(gtab, acc[ks][2]),
                                          sgelu(gtab, acc[ks][3]));
                const uint32_t hi = fp8x4(sgelu(gtab, acc[ks][4]), sgelu(gtab, acc[ks][5]), sgelu(gtab, acc[ks][6]),
                                          sgelu(gtab, acc[ks][7]));
                af[ks] = (long)(((uint64_t)hi << 32) | lo);
            } else {
#pragma unroll
                for (int j = 0; j < 8; j++) af[ks][j] = (__bf16)sgelu(gtab, acc[ks][j]);
            }
        }
        // layer 2 + output
        float part[4] = {0.f, 0.f, 0.f, 0.f};
        for (int nb = 0; nb < H / 16; nb++) {
            f32x4 a2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 8; ks++) {
                const AF b = *reinterpret_cast<const AF *>(w2s + (nb * 16 + c16) * WLD + 32 * ks + kq);
                if constexpr (kFp8)
                    a2 = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(af[ks], b, a2, 0, 0, 0);
                else
                    a2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks], b, a2, 0, 0, 0);
            }
            const float bb = w32[o.b2 + nb * 16 + c16], ww = w32[o.w3 + nb * 16 + c16];
#pragma unroll
            for (int i = 0; i < 4; i++) part[i] = fmaf(sgelu(gtab, fmaf(a2[i], inv2, bb)), ww, part[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; i++) part[i] = dpp_sum16(part[i]);
        if (c16 == 0) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int64_t kk = base + r0 + i;
                if (kk < end) pred[kk] = part[i] + w32[o.b3];
            }
        }
    }
}

// Combined first-layer rows C_t[p] = W1[(t + 1) N + p] + s_t W1[p] (FP64 sums, one rounding).
__global__ void k_refresh_combined(const double *__restrict__ w, int N, int H, float *__restrict__ cw1) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)4 * N * H) return;
    const int t = (int)(e / ((int64_t)N * H));
    const int64_t pu = e - (int64_t)t * N * H;  // p * H + u
    const double sgn = t < 2 ? -1.0 : 1.0;
    cw1[e] = (float)(w[(int64_t)(t + 1) * N * H + pu] + sgn * w[pu]);
}

// Per-tensor scale of the FP8 W2: the power of two 2^k with max|W2| 2^k <= 448
// (one block), then W2^T quantised to E4M3 (RNE, saturated).
__global__ void __launch_bounds__(256) k_w2_scale(const double *__restrict__ w, int N, int H,
                                                  float *__restrict__ scale2) {
    __shared__ double sh[256];
    const ScreenOff o = screen_off(N, H);
    double m = 0.0;
    for (int64_t e = threadIdx.x; e < (int64_t)H * H; e += 256) m = fmax(m, fabs(w[o.W2 + e]));
    sh[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        int k = 0;
        if (sh[0] > 0.0) k = (int)floor(log2(448.0 / sh[0]));
        if (k > 60) k = 60;
        if (k < -60) k = -60;
        scale2[0] = (float)ldexp(1.0, k);   // applied to W2 before quantisation
        scale2[1] = (float)ldexp(1.0, -k);  // applied to the products
    }
}

__global__ void k_w2_fp8(const double *__restrict__ w, int N, int H, const float *__restrict__ scale2,
                         uint8_t *__restrict__ w2f8) {
    const ScreenOff o = screen_off(N, H);
    const int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;  // four k of one n
    if (e >= (int64_t)H * H) return;
    const int nn = (int)(e / H), k = (int)(e % H);
    const float s = scale2[0];
    float v[4];
    for (int u = 0; u < 4; u++) v[u] = (float)w[o.W2 + (int64_t)(k + u) * H + nn] * s;
    *reinterpret_cast<uint32_t *>(w2f8 + e) = fp8x4(v[0], v[1], v[2], v[3]);
}

static unsigned gridfor(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

static nnqs_status ensure_scratch(nnqs_screen *s, size_t bytes, hipStream_t st) {
    if (s->scratch_bytes >= bytes) return NNQS_OK;
    NNQS_HIP_CHECK(hipStreamSynchronize(st));
    hipFree(s->scratch);
    s->scratch = nullptr;
    s->scratch_bytes = 0;
    if (hipMalloc(&s->scratch, bytes) != hipSuccess) return fail(NNQS_ENOMEM, "screen scratch of %zu bytes", bytes);
    s->scratch_bytes = bytes;
    return NNQS_OK;
}

nnqs_status screen_refresh(nnqs_screen *s, hipStream_t st) {
    if (!s->infer_dirty) return NNQS_OK;
    const ScreenOff o = screen_off(s->N, s->H);
    hipLaunchKernelGGL(k_refresh_infer, dim3(gridfor(o.total)), dim3(256), 0, st, s->w, s->N, s->H, s->w32, s->w2t);
    hipLaunchKernelGGL(k_refresh_combined, dim3(gridfor((int64_t)4 * s->N * s->H)), dim3(256), 0, st, s->w, s->N, s->H,
                       s->cw1);
    hipLaunchKernelGGL(k_w2_scale, dim3(1), dim3(256), 0, st, s->w, s->N, s->H, s->w2scale);
    hipLaunchKernelGGL(k_w2_fp8, dim3(gridfor((int64_t)s->H * s->H / 4)), dim3(256), 0, st, s->w, s->N, s->H,
                       (const float *)s->w2scale, s->w2f8);
    NNQS_HIP_CHECK(hipGetLastError());
    s->infer_dirty = false;
    return NNQS_OK;
}

// BF16 (or FP8) inference into FP32 predictions (used by the full local energy).
nnqs_status screen_infer(nnqs_screen *s, const uint64_t *keys, const uint8_t *exc, int64_t n, float *pred,
                         hipStream_t st, bool fp8) {
    if (s->H != kScreenH) return fail(NNQS_EUNSUPPORTED, "BF16 / FP8 screen inference needs hidden = 256");
    nnqs_status r = screen_refresh(s, st);
    if (r != NNQS_OK) return r;
    // one block of kScreenWaves waves per CU (W2 fills most of its LDS), each
    // wave a contiguous run of connections
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    int64_t blocks = (n + 32 * kScreenWaves - 1) / (32 * kScreenWaves);
    if (blocks > cus) blocks = cus;
    TimedRegion tr("k_screen_infer", st);
    if (fp8)
        hipLaunchKernelGGL(k_screen_infer<true>, dim3((unsigned)blocks), dim3(64 * kScreenWaves), 0, st, s->N, s->w32,
                           s->cw1, s->w2t, s->w2f8, (const float *)s->w2scale + 1, s->gelu_tab, keys, exc, n, pred);
    else
        hipLaunchKernelGGL(k_screen_infer<false>, dim3((unsigned)blocks), dim3(64 * kScreenWaves), 0, st, s->N,
                           s->w32, s->cw1, s->w2t, s->w2f8, (const float *)s->w2scale + 1, s->gelu_tab, keys, exc, n,
                           pred);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

// Sum of squared prediction errors, deterministic two-stage reduction:
// block partials (fixed per-thread strides, tree in LDS), then one block.
constexpr int kJudgeBlocks = 256;
__global__ void __launch_bounds__(256) k_sq_err_partial(const double *__restrict__ pred,
                                                        const double *__restrict__ target, int64_t n,
                                                        double *__restrict__ part) {
    __shared__ double sh[256];
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) {
        const double d = pred[k] - target[k];
        acc = fma(d, d, acc);
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void __launch_bounds__(256) k_sq_err_final(const double *__restrict__ part, int nb,
                                                      double *__restrict__ out) {
    __shared__ double sh[256];
    sh[threadIdx.x] = (int)threadIdx.x < nb ? part[threadIdx.x] : 0.0;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sh[0];
}

// Forward (and optionally the MSE gradient) in precision T.  Scratch holds
// z1, z2 ([n][H] each) and y ([n]), with the gradient a1, a2, d1, d2, gy and
// the partial sums of w3 ([16][H] FP64) too, and for FP32 a converted copy of
// the weights.
template <typename T>
static nnqs_status screen_fwd_bwd(nnqs_screen *s, const uint64_t *keys, const uint8_t *exc, const double *target,
                                  int64_t n, double *pred, double *grad, double *loss, hipStream_t st) {
    const int N = s->N, H = s->H;
    const ScreenOff o = screen_off(N, H);
    const size_t nh = (size_t)n * H, nw = sizeof(T) == 8 ? 0 : (size_t)o.total;
    const size_t np = grad ? (size_t)16 * H : 0;
    nnqs_status r =
        ensure_scratch(s, np * 8 + ((grad ? 6 : 2) * nh + 2 * (size_t)n + nw) * sizeof(T) + 256, st);
    if (r != NNQS_OK) return r;
    double *w3p = static_cast<double *>(s->scratch);
    T *z1 = reinterpret_cast<T *>(w3p + np), *z2 = z1 + nh, *y = z2 + nh, *gy = y + n, *wc = gy + n, *a1 = nullptr,
      *a2 = nullptr, *d1 = nullptr, *d2 = nullptr;
    if (grad) {
        a1 = wc + nw;
        a2 = a1 + nh;
        d1 = a2 + nh;
        d2 = d1 + nh;
    }
    const T *w;
    if constexpr (sizeof(T) == 8) {
        w = s->w;
    } else {
        hipLaunchKernelGGL(k_convert_f32, dim3(gridfor(o.total)), dim3(256), 0, st, s->w, wc, o.total);
        w = wc;
    }
    const unsigned ct = gridfor(H, 64);
    // a launch holds fewer than 2^32 threads, and these take up to 64 per example
    constexpr int64_t kMaxRows = (int64_t)1 << 24;
    for (int64_t k0 = 0; k0 < n; k0 += kMaxRows) {
        const int64_t m = std::min(kMaxRows, n - k0), h0 = k0 * H;
        T *a1k = a1 ? a1 + h0 : nullptr, *a2k = a2 ? a2 + h0 : nullptr;
        hipLaunchKernelGGL(k_screen_layer1<T>, dim3(gridfor(m, 4)), dim3(256), 0, st, N, H, w, keys + 2 * k0, exc + 4 * k0,
                           m, a1k, z1 + h0);
        hipLaunchKernelGGL((k_screen_hidden<T, false>), dim3(gridfor(m, 32), ct), dim3(256), 0, st, (const T *)(z1 + h0),
                           w + o.W2, w + o.b2, (const T *)nullptr, m, H, a2k, z2 + h0, (const T *)nullptr,
                           (const T *)nullptr, n, (double *)nullptr);
        hipLaunchKernelGGL(k_screen_out<T>, dim3(gridfor(m, 16)), dim3(256), 0, st, (const T *)a2k, (const T *)(z2 + h0), w,
                           N, H, m, n, grad ? target + k0 : nullptr, y + k0, pred ? pred + k0 : nullptr, gy + k0,
                           d2 ? d2 + h0 : nullptr);
    }
    if (grad) {
        for (int64_t k0 = 0; k0 < n; k0 += kMaxRows) {
            const int64_t m = std::min(kMaxRows, n - k0), h0 = k0 * H;
            const unsigned sums = k0 + m == n ? 16 : 0;  // the partial sums' blocks, once
            hipLaunchKernelGGL((k_screen_hidden<T, true>), dim3(gridfor(m, 32) + sums, ct), dim3(256), 0, st,
                               (const T *)(d2 + h0), w + o.W2, (const T *)nullptr, (const T *)(a1 + h0), m, H,
                               (T *)nullptr, d1 + h0, (const T *)z2, (const T *)gy, n, w3p);
        }
        const int jt = (H + 31) / 32, tiles = ((5 * N + 31) / 32 + jt) * jt;
        hipLaunchKernelGGL(k_screen_grads<T>, dim3((unsigned)(2 + tiles)), dim3(256), 0, st, N, H, keys, exc, target, n,
                           (const T *)z1, (const T *)d1, (const T *)d2, (const T *)y, (const T *)gy,
                           (const double *)w3p, grad, loss);
    }
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

}  // namespace nnqs

using namespace nnqs;

extern "C" {

int64_t nnqs_screen_weight_count(int32_t n_spin_orb, int32_t hidden) {
    if (n_spin_orb < 4 || n_spin_orb > 128 || (n_spin_orb & 1) || hidden < 1 || hidden > 1024) return -1;
    return screen_off(n_spin_orb, hidden).total;
}

nnqs_status nnqs_screen_create(nnqs_screen **out, int32_t n_spin_orb, int32_t hidden, const double *weights) {
    clear_error();
    if (!out || !weights) return fail(NNQS_EINVAL, "null pointer argument");
    *out = nullptr;
    const int64_t cnt = nnqs_screen_weight_count(n_spin_orb, hidden);
    if (cnt < 0) return fail(NNQS_EINVAL, "invalid screen shape (N=%d, hidden=%d)", n_spin_orb, hidden);
    nnqs_screen *s = new nnqs_screen();
    s->N = n_spin_orb;
    s->H = hidden;
    s->count = cnt;
    if (hipMalloc(&s->w, cnt * 8) != hipSuccess || hipMalloc(&s->m, cnt * 8) != hipSuccess ||
        hipMalloc(&s->v, cnt * 8) != hipSuccess || hipMalloc(&s->w32, cnt * 4) != hipSuccess ||
        hipMalloc(&s->w2t, (size_t)hidden * hidden * 2) != hipSuccess ||
        hipMalloc(&s->cw1, (size_t)4 * n_spin_orb * hidden * 4) != hipSuccess ||
        hipMalloc(&s->w2f8, (size_t)hidden * hidden) != hipSuccess || hipMalloc(&s->w2scale, 2 * 4) != hipSuccess ||
        hipMalloc(&s->gelu_tab, 2 * kSGeluN * 4) != hipSuccess) {
        nnqs_screen_destroy(s);
        return fail(NNQS_ENOMEM, "screen allocation failed");
    }
    std::vector<float> gt(2 * kSGeluN);
    for (int i = 0; i < kSGeluN; i++) {  // Phi at the knots, in FP64
        const double v0 = (i - (double)kSGeluOff) / kSGeluScale, v1 = v0 + 1.0 / kSGeluScale;
        const double p0 = 0.5 * std::erfc(-v0 / std::sqrt(2.0)), p1 = 0.5 * std::erfc(-v1 / std::sqrt(2.0));
        gt[2 * i] = (float)p0;
        gt[2 * i + 1] = (float)(p1 - p0);
    }
    if (hipMemcpy(s->gelu_tab, gt.data(), gt.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(s->w, weights, cnt * 8, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(s->m, 0, cnt * 8) != hipSuccess || hipMemset(s->v, 0, cnt * 8) != hipSuccess ||
        hipDeviceSynchronize() != hipSuccess) {
        nnqs_screen_destroy(s);
        return fail(NNQS_EHIP, "screen initialisation failed");
    }
    *out = s;
    return NNQS_OK;
}

nnqs_status nnqs_screen_destroy(nnqs_screen *s) {
    if (!s) return NNQS_OK;
    hipFree(s->w);
    hipFree(s->m);
    hipFree(s->v);
    hipFree(s->w32);
    hipFree(s->w2t);
    hipFree(s->cw1);
    hipFree(s->w2f8);
    hipFree(s->w2scale);
    hipFree(s->gelu_tab);
    hipFree(s->scratch);
    hipFree(s->jscratch);
    delete s;
    return NNQS_OK;
}

nnqs_status nnqs_screen_get_weights(const nnqs_screen *s, double *host_out, void *stream) {
    clear_error();
    if (!s || !host_out) return fail(NNQS_EINVAL, "null pointer argument");
    hipStream_t st = as_stream(stream);
    NNQS_HIP_CHECK(hipMemcpyAsync(host_out, s->w, s->count * 8, hipMemcpyDeviceToHost, st));
    NNQS_HIP_CHECK(hipStreamSynchronize(st));
    return NNQS_OK;
}

nnqs_status nnqs_screen_get_state(const nnqs_screen *s, double *m_out, double *v_out, int64_t *t_out,
                                  void *stream) {
    clear_error();
    if (!s || !m_out || !v_out || !t_out) return fail(NNQS_EINVAL, "null pointer argument");
    hipStream_t st = as_stream(stream);
    NNQS_HIP_CHECK(hipMemcpyAsync(m_out, s->m, s->count * 8, hipMemcpyDeviceToHost, st));
    NNQS_HIP_CHECK(hipMemcpyAsync(v_out, s->v, s->count * 8, hipMemcpyDeviceToHost, st));
    NNQS_HIP_CHECK(hipStreamSynchronize(st));
    *t_out = s->t;
    return NNQS_OK;
}

nnqs_status nnqs_screen_set_state(nnqs_screen *s, const double *m, const double *v, int64_t t, void *stream) {
    clear_error();
    if (!s || !m || !v) return fail(NNQS_EINVAL, "null pointer argument");
    if (t < 0) return fail(NNQS_EINVAL, "negative Adam step count");
    hipStream_t st = as_stream(stream);
    NNQS_HIP_CHECK(hipMemcpyAsync(s->m, m, s->count * 8, hipMemcpyHostToDevice, st));
    NNQS_HIP_CHECK(hipMemcpyAsync(s->v, v, s->count * 8, hipMemcpyHostToDevice, st));
    NNQS_HIP_CHECK(hipStreamSynchronize(st));
    s->t = t;
    return NNQS_OK;
}

nnqs_status nnqs_screen_forward(nnqs_screen *s, const uint64_t *keys, const uint8_t *exc, int64_t n,
                                int32_t precision, double *pred, void *stream) {
    clear_error();
    if (!s || !keys || !exc || !pred) return fail(NNQS_EINVAL, "null pointer argument");
    if (n <= 0) return fail(NNQS_EINVAL, "n must be positive");
    hipStream_t st = as_stream(stream);
    if (precision == NNQS_FP64) return screen_fwd_bwd<double>(s, keys, exc, nullptr, n, pred, nullptr, nullptr, st);
    if (precision == NNQS_FP32) return screen_fwd_bwd<float>(s, keys, exc, nullptr, n, pred, nullptr, nullptr, st);
    if (precision == NNQS_BF16 || precision == NNQS_FP8) {
        nnqs_status r = ensure_scratch(s, (size_t)n * 4 + 256, st);
        if (r != NNQS_OK) return r;
        float *p32 = static_cast<float *>(s->scratch);
        r = screen_infer(s, keys, exc, n, p32, st, precision == NNQS_FP8);
        if (r != NNQS_OK) return r;
        hipLaunchKernelGGL(k_to_double<float>, dim3(gridfor(n)), dim3(256), 0, st, p32, pred, n);
        NNQS_HIP_CHECK(hipGetLastError());
        return NNQS_OK;
    }
    return fail(NNQS_EUNSUPPORTED, "unknown precision %d", precision);
}

nnqs_status nnqs_screen_gradient(nnqs_screen *s, const uint64_t *keys, const uint8_t *exc, const double *target,
                                 int64_t n, int32_t precision, double *grad, double *loss, void *stream) {
    clear_error();
    if (!s || !keys || !exc || !target || !grad) return fail(NNQS_EINVAL, "null pointer argument");
    if (n <= 0) return fail(NNQS_EINVAL, "n must be positive");
    hipStream_t st = as_stream(stream);
    if (precision == NNQS_FP64) return screen_fwd_bwd<double>(s, keys, exc, target, n, nullptr, grad, loss, st);
    if (precision == NNQS_FP32) return screen_fwd_bwd<float>(s, keys, exc, target, n, nullptr, grad, loss, st);
    return fail(NNQS_EUNSUPPORTED, "gradients are available in FP64 and FP32");
}

nnqs_status nnqs_screen_adam_step(nnqs_screen *s, const double *grad, double lr, double beta1, double beta2,
                                  double eps, void *stream) {
    clear_error();
    if (!s || !grad) return fail(NNQS_EINVAL, "null pointer argument");
    if (!(lr > 0.0) || !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps > 0.0))
        return fail(NNQS_EINVAL, "invalid Adam hyper-parameters");
    hipStream_t st = as_stream(stream);
    s->t += 1;
    const double c1 = 1.0 - std::pow(beta1, (double)s->t), c2 = 1.0 - std::pow(beta2, (double)s->t);
    hipLaunchKernelGGL(k_adam, dim3(gridfor(s->count)), dim3(256), 0, st, s->w, grad, s->m, s->v, s->count, lr, beta1,
                       beta2, eps, c1, c2);
    NNQS_HIP_CHECK(hipGetLastError());
    s->infer_dirty = true;
    return NNQS_OK;
}


nnqs_status nnqs_screen_judge(nnqs_screen *s, const uint64_t *xkeys, const uint8_t *exc, const double *target,
                              int64_t n, int32_t precision, double max_rmse, double *rmse, int32_t *usable,
                              void *stream) {
    clear_error();
    if (!s || !xkeys || !exc || !target || !rmse) return fail(NNQS_EINVAL, "null pointer argument");
    if (n <= 0) return fail(NNQS_EINVAL, "n must be positive");
    if (!(max_rmse >= 0.0)) return fail(NNQS_EINVAL, "max_rmse must be >= 0");
    hipStream_t st = as_stream(stream);
    const size_t need = ((size_t)n + kJudgeBlocks + 1) * sizeof(double);
    if (s->jscratch_bytes < need) {
        NNQS_HIP_CHECK(hipStreamSynchronize(st));
        hipFree(s->jscratch);
        s->jscratch = nullptr;
        s->jscratch_bytes = 0;
        if (hipMalloc(&s->jscratch, need) != hipSuccess) return fail(NNQS_ENOMEM, "judge scratch of %zu bytes", need);
        s->jscratch_bytes = need;
    }
    double *pred = static_cast<double *>(s->jscratch), *part = pred + n, *sum = part + kJudgeBlocks;
    const nnqs_status r = nnqs_screen_forward(s, xkeys, exc, n, precision, pred, stream);
    if (r != NNQS_OK) return r;
    const int nb = (int)std::min<int64_t>(kJudgeBlocks, (n + 255) / 256);
    hipLaunchKernelGGL(k_sq_err_partial, dim3(nb), dim3(256), 0, st, (const double *)pred, target, n, part);
    hipLaunchKernelGGL(k_sq_err_final, dim3(1), dim3(256), 0, st, (const double *)part, nb, sum);
    NNQS_HIP_CHECK(hipGetLastError());
    double total = 0.0;
    NNQS_HIP_CHECK(hipMemcpyAsync(&total, sum, 8, hipMemcpyDeviceToHost, st));
    NNQS_HIP_CHECK(hipStreamSynchronize(st));
    *rmse = std::sqrt(total / (double)n);
    if (usable) *usable = *rmse <= max_rmse ? 1 : 0;
    return NNQS_OK;
}

}  // extern "C"
