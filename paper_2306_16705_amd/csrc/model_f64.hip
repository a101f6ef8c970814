// The FP64 network: entry points (the transformer in one launch,
// transformer_f64.hip; the phase MLP of Section 4.1 here), and the layer-wise
// kernels of the gradient's forward, which keeps every activation: LayerNorm
// one wave per row, the dense layers an LDS-tiled FP64 MFMA product (64 x 64
// output tile per block) with bias, GELU or residual-add epilogues, causal
// attention on FP64 MFMA one block per (configuration, head).  Only the
// summation order differs from a one-configuration-at-a-time evaluation.
#include <cmath>

#include "f64_kernels.hpp"

namespace nnqs {

constexpr int64_t kF64Batch = 4096;  // configurations per pass

// Tokens (previous-token input) and embeddings: h[b*K + s][c].
__global__ void k64_embed(ModelView M, const uint64_t *__restrict__ keys, int64_t B, int8_t *__restrict__ tok,
                          double *__restrict__ h) {
    const int K = M.K, d = M.d;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= B * K * d) return;
    const int64_t row = e / d;
    const int c = (int)(e - row * d);
    const int64_t b = row / K;
    const int s = (int)(row - b * K);
    Key x;
    x.lo = keys[2 * b];
    x.hi = keys[2 * b + 1];
    auto token = [&](int pos) {
        const int i = K - 1 - pos;  // position s holds spatial orbital K-1-s
        return key_bit(x, 2 * i) + 2 * key_bit(x, 2 * i + 1);
    };
    if (c == 0) tok[row] = (int8_t)token(s);
    const int prev = s == 0 ? 4 : token(s - 1);
    h[e] = M.w64[M.off.tok_emb + prev * d + c] + M.w64[M.off.pos_emb + (int64_t)s * d + c];
}

// LayerNorm (eps 1e-5) of rows of width 64: one wave per row, lane = column.
__global__ void __launch_bounds__(256) k64_layernorm(const double *__restrict__ in, const double *__restrict__ g,
                                                     const double *__restrict__ b, int64_t rows,
                                                     double *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const double v = in[row * 64 + lane];
    double s = v;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    const double mean = s / 64.0;
    double q = (v - mean) * (v - mean);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) q += __shfl_xor(q, off, 64);
    const double r = 1.0 / sqrt(q / 64.0 + 1e-5);
    out[row * 64 + lane] = (v - mean) * r * g[lane] + b[lane];
}

// C[r][j] = epi(bias[j] + sum_k A[r][k] B[k][j]) for r < M, j < N, with
// B[k][j] = W[k][j], or W[j][k] with TB (products with a transposed weight in
// the backward).  Block: TM x 64 tile of C, four waves: 16 rows each by all 64
// columns (TM = 64), or 16 rows by 32 columns (TM = 32), on
// v_mfma_f64_16x16x4_f64 (lane l holds A[l & 15][l >> 4] and B[l >> 4][l & 15];
// accumulator register i of lane l holds row (l >> 4) + 4 i, column l & 15);
// k in slices of 32 through LDS, the next slice's global loads in flight
// during the current slice's products.  Rows of 36 and 80 doubles put the 32
// lanes of half a wave on 64 different banks for both operands (rows of 33
// and 65 gave two-way conflicts).
// EPI 0 stores, 2 stores GELU, 3 stores GELU' and, in C2, GELU, 4 stores the
// sum times U (a GELU' of the forward), 5 stores src + the sum.

template <int TM>
struct GemmLds {
    double As[TM][36];
    double Ws[32][80];
};

// The products of one K x 64 weight (ldw columns) with A's rows, added to acc.
template <int TM, bool TB>
__device__ __forceinline__ void gemm64_acc(GemmLds<TM> &S, f64x4 (&acc)[TM / 16], const double *__restrict__ A, int lda,
                                           const double *__restrict__ W, int ldw, int64_t M, int N, int Kd, int c0) {
    constexpr int EA = TM / 8, NC = TM / 16;  // A elements per thread and slice; column tiles per wave
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lr = l & 15, lk = l >> 4;
    const int rw = TM == 64 ? 16 * w : 16 * (w & 1), cw = TM == 64 ? 0 : 32 * (w >> 1);
    const int64_t r0 = (int64_t)blockIdx.y * TM;
    // slice loads: thread t takes A[r0 + (t >> 5) + 8 e][k0 + (t & 31)] and
    // W[k0 + (t >> 6) + 4 e][c0 + (t & 63)] (coalesced rows); with TB,
    // W[c0 + (t >> 5) + 8 e][k0 + (t & 31)] into the slice's column
    const int at = threadIdx.x & 31, ar = threadIdx.x >> 5, wc = threadIdx.x & 63, wr = threadIdx.x >> 6;
    double pa[EA], pw[8];
    auto load = [&](int k0) {
#pragma unroll
        for (int e = 0; e < EA; e++) {
            const int64_t r = r0 + ar + 8 * e;
            pa[e] = (r < M && k0 + at < Kd) ? A[r * lda + k0 + at] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < 8; e++) {
            if (TB) {
                const int cc = c0 + ar + 8 * e;
                pw[e] = (cc < N && k0 + at < Kd) ? W[(int64_t)cc * ldw + k0 + at] : 0.0;
            } else {
                const int kw = k0 + wr + 4 * e;
                pw[e] = (kw < Kd && c0 + wc < N) ? W[(int64_t)kw * ldw + c0 + wc] : 0.0;
            }
        }
    };
    load(0);
    for (int k0 = 0; k0 < Kd; k0 += 32) {
        __syncthreads();  // the previous slice is consumed
#pragma unroll
        for (int e = 0; e < EA; e++) S.As[ar + 8 * e][at] = pa[e];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            if (TB) S.Ws[at][ar + 8 * e] = pw[e];
            else S.Ws[wr + 4 * e][wc] = pw[e];
        }
        __syncthreads();
        if (k0 + 32 < Kd) load(k0 + 32);  // the next slice's loads overlap this slice's products
#pragma unroll
        for (int k4 = 0; k4 < 32; k4 += 4) {
            const double a = S.As[rw + lr][k4 + lk];
#pragma unroll
            for (int cb = 0; cb < NC; cb++)
                acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, S.Ws[k4 + lk][cw + cb * 16 + lr], acc[cb], 0, 0, 0);
        }
    }
}

template <int TM, int EPI>
__device__ __forceinline__ void gemm64_store(const f64x4 (&acc)[TM / 16], const double *__restrict__ bias, int64_t M,
                                             int N, double *__restrict__ C, int ldc, int c0, const GemmEpi &E) {
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lr = l & 15, lk = l >> 4;
    const int rw = TM == 64 ? 16 * w : 16 * (w & 1), cw = TM == 64 ? 0 : 32 * (w >> 1);
    const int64_t r0 = (int64_t)blockIdx.y * TM;
#pragma unroll
    for (int cb = 0; cb < TM / 16; cb++) {
        const int c = c0 + cw + cb * 16 + lr;
        if (c >= N) continue;
        const double bc = bias ? bias[c] : 0.0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t r = r0 + rw + lk + 4 * i;
            if (r >= M) continue;
            const double v = bc + acc[cb][i];
            double *dst = C + r * ldc + c;
            if (EPI == 2) *dst = gelu_f64(v);
            else if (EPI == 3) {
                const double cdf = 0.5 * (1.0 + erf(v * 0.70710678118654752440));
                *dst = cdf + v * (0.39894228040143267794 * exp(-0.5 * v * v));
                E.C2[r * ldc + c] = v * cdf;
            } else if (EPI == 4) *dst = v * E.U[r * ldc + c];
            else if (EPI == 5) *dst = E.src[r * ldc + c] + v;
            else *dst = v;
        }
    }
}

// At least four waves per SIMD: the register budget that sets holds the tile
// without spills.
template <int EPI, bool TB, int TM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k64_gemm(const double *__restrict__ A, int lda, const double *__restrict__ W, int ldw, const double *__restrict__ bias,
         int64_t M, int N, int Kd, double *__restrict__ C, int ldc, GemmEpi E) {
    __shared__ GemmLds<TM> S;
    f64x4 acc[TM / 16] = {};
    gemm64_acc<TM, TB>(S, acc, A, lda, W, ldw, M, N, Kd, blockIdx.x * 64);
    gemm64_store<TM, EPI>(acc, bias, M, N, C, ldc, blockIdx.x * 64, E);
}

// Rows per tile: 64, or 32 where 64-row tiles would leave CUs without a block
// (7,680 rows by 64 columns: 120 blocks against 240; the residual product
// 11.3 against 17.3 us, and 7,680 by 256 of depth 64, 480 against 960,
// 24 against 28 us).  Beyond that both measure the same within 0.2 % (the
// phase products of 4.3 ms of local energies) and 64 read the weights half as
// often.
static bool small_tiles(int64_t M, int N) { return ((M + 63) / 64) * ((N + 63) / 64) < 512; }

template <int EPI, bool TB>
void gemm64(const double *A, int lda, const double *W, int ldw, const double *bias, int64_t M, int N, int Kd, double *C,
            int ldc, const GemmEpi &E, hipStream_t st) {
    const unsigned gx = (unsigned)((N + 63) / 64);
    if (small_tiles(M, N))
        hipLaunchKernelGGL((k64_gemm<EPI, TB, 32>), dim3(gx, (unsigned)((M + 31) / 32)), dim3(256), 0, st, A, lda, W, ldw,
                           bias, M, N, Kd, C, ldc, E);
    else
        hipLaunchKernelGGL((k64_gemm<EPI, TB, 64>), dim3(gx, (unsigned)((M + 63) / 64)), dim3(256), 0, st, A, lda, W, ldw,
                           bias, M, N, Kd, C, ldc, E);
}

// Q, K and V of the same rows in one launch: column block x = 0, 1, 2 of the
// grid takes the weight and bias at W + x ws, bias + x ws (the layer block
// keeps W_q, b_q, W_k, b_k, W_v, b_v at equal strides) and writes C + x cs.
template <int TM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k64_gemm_qkv(const double *__restrict__ a, const double *__restrict__ W, const double *__restrict__ bias, int64_t ws,
             int64_t M, double *__restrict__ C, int64_t cs) {
    __shared__ GemmLds<TM> S;
    const int x = blockIdx.x;
    f64x4 acc[TM / 16] = {};
    gemm64_acc<TM, false>(S, acc, a, 64, W + x * ws, 64, M, 64, 64, 0);
    gemm64_store<TM, 0>(acc, bias + x * ws, M, 64, C + x * cs, 64, 0, GemmEpi{});
}

void gemm64_qkv(const double *a, const double *W, const double *bias, int64_t ws, int64_t M, double *C, int64_t cs,
                hipStream_t st) {
    if (small_tiles(M, 192))
        hipLaunchKernelGGL(k64_gemm_qkv<32>, dim3(3, (unsigned)((M + 31) / 32)), dim3(256), 0, st, a, W, bias, ws, M, C,
                           cs);
    else
        hipLaunchKernelGGL(k64_gemm_qkv<64>, dim3(3, (unsigned)((M + 63) / 64)), dim3(256), 0, st, a, W, bias, ws, M, C,
                           cs);
}

// The transpose of that: C = sum_x A_x W_x^T, A_x = A + x as, W_x = W + x ws.
template <int TM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k64_gemm_res(const double *__restrict__ A, int64_t as, const double *__restrict__ W, int64_t ws, int64_t M,
             double *__restrict__ C) {
    __shared__ GemmLds<TM> S;
    f64x4 acc[TM / 16] = {};
    for (int x = 0; x < 3; x++) gemm64_acc<TM, true>(S, acc, A + x * as, 64, W + x * ws, 64, M, 64, 64, 0);
    gemm64_store<TM, 0>(acc, nullptr, M, 64, C, 64, 0, GemmEpi{});
}

void gemm64_qkv_back(const double *A, int64_t as, const double *W, int64_t ws, int64_t M, double *C, hipStream_t st) {
    if (small_tiles(M, 64))
        hipLaunchKernelGGL(k64_gemm_res<32>, dim3(1, (unsigned)((M + 31) / 32)), dim3(256), 0, st, A, as, W, ws, M, C);
    else
        hipLaunchKernelGGL(k64_gemm_res<64>, dim3(1, (unsigned)((M + 63) / 64)), dim3(256), 0, st, A, as, W, ws, M, C);
}

// Causal attention on FP64 MFMA: one block per (configuration, head), wave w
// its queries 16 w .. 16 w + 15; q, k, v and the output are [B*K][64] with
// head hh in columns 16 hh .. 16 hh + 15.  Per wave:
// S = Q K^T in 16 x 16 x 4 tiles (accumulator register i of lane l holds
// query (l >> 4) + 4 i, key l & 15 of the tile), the softmax of each query
// row over the 16 lanes that hold it (the largest score, then one
// exponential per key), P through LDS into the A-operand layout, O = P V.
// Rows at or beyond K read as zero and are never written.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k64_attention(const double *__restrict__ q, const double *__restrict__ k, const double *__restrict__ v, int K,
              double scale, double *__restrict__ o) {
    __shared__ double Ps[4][16][64 + 1];
    const int l = threadIdx.x & 63, qb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = l & 15, lk = l >> 4;
    if (16 * qb >= K) return;  // wave-uniform; the kernel has no block barrier
    const int64_t base = (int64_t)(blockIdx.x >> 2) * K * 64 + (blockIdx.x & 3) * 16;
    const double *qh = q + base, *kh = k + base, *vh = v + base;
    const double c2 = scale * 1.4426950408889634;  // the softmax in base 2
    ConstF64 *tab = exp2_table();
    // Four adjacent head columns of row s (lane lk's share of the score
    // product's contraction, column 4 lk + k4): one 32-byte load.
    auto ld4 = [&](const double *p, int s) {
        return s < K ? *reinterpret_cast<const f64x4 *>(p + (int64_t)s * 64 + 4 * lk) : f64x4{0.0, 0.0, 0.0, 0.0};
    };
    double(*P)[64 + 1] = Ps[qb];
    const f64x4 qf = ld4(qh, qb * 16 + lr);
    f64x4 st[4], vf[4];  // scores; V[16 kb + 4 i + lk][lr]
#pragma unroll
    for (int kb = 0; kb < 4; kb++) {
        st[kb] = f64x4{0.0, 0.0, 0.0, 0.0};
        if (kb > qb) continue;
        const f64x4 kf = ld4(kh, kb * 16 + lr);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int s = 16 * kb + 4 * i + lk;
            vf[kb][i] = s < K ? vh[(int64_t)s * 64 + lr] : 0.0;
            st[kb] = __builtin_amdgcn_mfma_f64_16x16x4f64(qf[i], kf[i], st[kb], 0, 0, 0);
        }
    }
    // key 16 kb + lr is visible to query 16 qb + lk + 4 i when kb < qb, or kb == qb and lr <= lk + 4 i
#pragma unroll
    for (int i = 0; i < 4; i++) {
        double mx = -INFINITY, den = 0.0;
#pragma unroll
        for (int kb = 0; kb < 4; kb++)
            if (kb < qb || (kb == qb && lr <= lk + 4 * i)) mx = fmax(mx, st[kb][i]);
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 16));
#pragma unroll
        for (int kb = 0; kb < 4; kb++) {
            if (kb > qb) continue;
            const double p = kb < qb || lr <= lk + 4 * i ? exp2_f64(tab, (st[kb][i] - mx) * c2) : 0.0;
            st[kb][i] = p;
            den += p;
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) den += __shfl_xor(den, off, 16);
        const double rden = 1.0 / den;
#pragma unroll
        for (int kb = 0; kb < 4; kb++)
            if (kb <= qb) P[lk + 4 * i][kb * 16 + lr] = st[kb][i] * rden;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    f64x4 ot = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kb = 0; kb < 4; kb++) {
        if (kb > qb) continue;
#pragma unroll
        for (int i = 0; i < 4; i++)
            ot = __builtin_amdgcn_mfma_f64_16x16x4f64(P[lr][16 * kb + 4 * i + lk], vf[kb][i], ot, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int s = qb * 16 + lk + 4 * i;
        if (s < K) o[base + (int64_t)s * 64 + lr] = ot[i];
    }
}

// Output head with the logit bias, the mask (Eq. 12, read with the lower
// bound too) and the log-probability of the actual token: one wave per
// (config, position).
__global__ void __launch_bounds__(256) k64_head(ModelView M, const double *__restrict__ a,
                                                const int8_t *__restrict__ tok, int64_t B, double *__restrict__ lp) {
    // lane = model column (d = 64)
    const int K = M.K;
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= B * K) return;  // wave-uniform
    const int64_t b = row / K;
    const int s = (int)(row - b * K);
    // electrons placed before position s (lanes r < s hold token r)
    const int tr = lane < s ? tok[b * K + lane] : 0;
    const int up = __popcll(__ballot(tr & 1)), dn = __popcll(__ballot(tr >> 1));
    const double *W = M.w64;
    const double av = a[row * 64 + lane];
    double z[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
        double v = av * W[M.off.head_w + lane * 4 + t];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        z[t] = v;
    }
    if (lane != 0) return;
    const int rem = K - 1 - s, orb = K - 1 - s;
    bool ok[4];
    double mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        z[t] += W[M.off.head_b + t] + W[M.off.bias + orb * 4 + t];
        const int bu = t & 1, bd = t >> 1;
        ok[t] = (up + bu <= M.n_up) && (dn + bd <= M.n_dn) && (M.n_up - up - bu <= rem) && (M.n_dn - dn - bd <= rem);
        if (ok[t] && z[t] > mx) mx = z[t];
    }
    double den = 0.0;
#pragma unroll
    for (int t = 0; t < 4; t++)
        if (ok[t]) den += exp(z[t] - mx);
    const int ts = tok[row];
    lp[row] = ok[ts] ? (z[ts] - mx) - log(den) : -INFINITY;
}

// First phase layer from the occupation bits: z1[b][j] = GELU(b1[j] + sum
// over set bits p of W1[p][j]); configuration b is keys[b], or keys[list[b]].
__global__ void k64_phase1(ModelView M, const uint64_t *__restrict__ keys, const int32_t *__restrict__ list, int64_t B,
                           double *__restrict__ z1) {
    const int P = M.P;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= B * P) return;
    const int64_t b = e / P;
    const int j = (int)(e - b * P);
    const int64_t kb = list ? list[b] : b;
    Key x;
    x.lo = keys[2 * kb];
    x.hi = keys[2 * kb + 1];
    double acc = M.w64[M.off.ph_b1 + j];
    for (int p = 0; p < 2 * M.K; p++)
        if (key_bit(x, p)) acc += M.w64[M.off.ph_w1 + (int64_t)p * P + j];
    z1[e] = gelu_f64(acc);
}

// Phase of each configuration, b3 + z2 . w3 (one wave each, fixed-order lane
// sums), to phase[b] or phase[list[b]].
__global__ void __launch_bounds__(256) k64_phase_out(ModelView M, const double *__restrict__ z2,
                                                     const int32_t *__restrict__ list, int64_t B,
                                                     double *__restrict__ phase) {
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (b >= B) return;
    double ph = 0.0;
    for (int i = lane; i < M.P; i += 64) ph += z2[b * M.P + i] * M.w64[M.off.ph_w3 + i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ph += __shfl_xor(ph, off, 64);
    if (lane == 0) phase[list ? list[b] : b] = M.w64[M.off.ph_b3] + ph;
}

// Per configuration: log|psi| = 1/2 sum_s lp, phase = b3 + z2 . w3 (one wave
// each, fixed-order lane sums).
__global__ void __launch_bounds__(256) k64_finish(ModelView M, const double *__restrict__ lp,
                                                  const double *__restrict__ z2, int64_t B,
                                                  double *__restrict__ logabs, double *__restrict__ phase) {
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (b >= B) return;
    double s = 0.0;
    for (int t = lane; t < M.K; t += 64) s += lp[b * M.K + t];
    double ph = 0.0;
    for (int i = lane; i < M.P; i += 64) ph += z2[b * M.P + i] * M.w64[M.off.ph_w3 + i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        s += __shfl_xor(s, off, 64);
        ph += __shfl_xor(ph, off, 64);
    }
    if (lane == 0) {
        logabs[b] = 0.5 * s;
        phase[b] = M.w64[M.off.ph_b3] + ph;
    }
}

// Causal attention backward on FP64 MFMA, one block per (configuration, head);
// q, k, v, o, dout (dO) and the outputs are [B*K][64] with head hh in columns
// 16 hh .. 16 hh + 15.  Three passes over the 16 x 16 tiles at or below the
// diagonal, wave w taking query block w in the first two and key block w in the
// third (at most five tiles a wave of the last two): the softmax's
// maximum and denominator and D = dO . O of every query; dQ^T += K^T dS^T per
// query block; dV^T += dO^T P and dK^T += Q^T dS per key block, with
//   P^T = exp(scale (K Q^T - max)) / den,  dS^T = P^T o (V dO^T - D)
// formed again in each (28 matrix instructions a tile in all: against keeping
// every dQ tile through one pass, that holds four waves per SIMD without
// spills).  Transposed tiles hold a query per lane (lr) and keys lk + 4 i, the
// operand of the dQ product as they are; the other two contract over queries
// and take P and dS through LDS.  Rows at or beyond K read as zero and are
// never written.  A wave per (configuration, head), all blocks one after another,
// left half the CUs without work at 128 configurations of K = 60: 68 us a layer,
// now 30.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k64x_attention_back(const double *__restrict__ q, const double *__restrict__ k, const double *__restrict__ v,
                    const double *__restrict__ o, const double *__restrict__ dout, int K, double scale,
                    double *__restrict__ dq, double *__restrict__ dk, double *__restrict__ dv) {
    __shared__ double Tl[4][2][16][18];  // P and dS of one tile, [query][key]
    __shared__ double St[3][64];         // max, 1 / den, D of every query
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = l & 15, lk = l >> 4;
    const int64_t base = (int64_t)(blockIdx.x >> 2) * K * 64 + (blockIdx.x & 3) * 16;
    // The lane's row is made anew in every pass of the loops below: loads that
    // do not change with the pass would otherwise all be held in registers.
    int lx = lr;
    auto rowop = [&](const double *p, int blk) -> f64x4 {  // lane lr: row 16 blk + lr, columns 4 lk ..
        const int s = 16 * blk + lx;
        return s < K ? *reinterpret_cast<const f64x4 *>(p + base + (int64_t)s * 64 + 4 * lk) : f64x4{0.0, 0.0, 0.0, 0.0};
    };
    auto colop = [&](const double *p, int blk, int i) -> double {  // row 16 blk + 4 i + lk, column lr
        const int s = 16 * blk + 4 * i + lk;
        return s < K ? p[base + (int64_t)s * 64 + lx] : 0.0;
    };
    auto tile = [&](const f64x4 &a, const f64x4 &b) -> f64x4 {  // a's rows by b's rows, contracted over the 16 columns
        f64x4 t = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < 4; i++) t = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[i], t, 0, 0, 0);
        return t;
    };
    auto xsum = [](double x) {
        x += __shfl_xor(x, 16, 64);
        return x + __shfl_xor(x, 32, 64);
    };
    auto sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const int nb = (K + 15) >> 4;
    const double c2 = scale * 1.4426950408889634;  // the softmax in base 2
    if (w < nb) {
        const int j = w;
        ConstF64 *tab = exp2_table();
        const f64x4 qf = rowop(q, j), gf = rowop(dout, j), of = rowop(o, j);
        double D = 0.0;
#pragma unroll
        for (int i = 0; i < 4; i++) D += gf[i] * of[i];
        D = xsum(D);
        // running maximum and denominator of the lane's keys, then of the four lanes
        double mx = -INFINITY, den = 0.0;
#pragma unroll 1
        for (int kb = 0; kb <= j; kb++) {
            asm volatile("" : "+v"(lx));
            const f64x4 st = tile(rowop(k, kb), qf);
            bool in[4];
            double m = mx;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                in[i] = kb < j || lk + 4 * i <= lr;
                m = in[i] ? fmax(m, st[i]) : m;
            }
            den *= m > mx ? exp2_f64(tab, (mx - m) * c2) : 1.0;
            mx = m;
#pragma unroll
            for (int i = 0; i < 4; i++) den += in[i] ? exp2_f64(tab, (st[i] - m) * c2) : 0.0;
        }
        double ml = fmax(mx, __shfl_xor(mx, 16, 64));
        ml = fmax(ml, __shfl_xor(ml, 32, 64));
        den = xsum(den > 0.0 ? den * exp2_f64(tab, (mx - ml) * c2) : den);
        mx = ml;
        if (lk == 0) {
            St[0][16 * j + lr] = mx;
            St[1][16 * j + lr] = 1.0 / den;
            St[2][16 * j + lr] = D;
        }
    }
    __syncthreads();  // every query's statistics; no block barrier follows
    if (w >= nb) return;
    // P^T and dS^T of one tile
    auto grads = [&](ConstF64 *tab, int j, int kb, f64x4 &p, f64x4 &ds) {
        p = tile(rowop(k, kb), rowop(q, j));
        const f64x4 dp = tile(rowop(v, kb), rowop(dout, j));
        const double mx = St[0][16 * j + lr], rden = St[1][16 * j + lr], D = St[2][16 * j + lr];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            p[i] = kb == j && lk + 4 * i > lr ? 0.0 : exp2_f64(tab, (p[i] - mx) * c2) * rden;
            ds[i] = p[i] * (dp[i] - D);
        }
    };
    {
        const int j = w;
        ConstF64 *tab = exp2_table();
        f64x4 dqt = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int kb = 0; kb <= j; kb++) {
            asm volatile("" : "+v"(lx));
            f64x4 p, ds;
            grads(tab, j, kb, p, ds);
#pragma unroll
            for (int i = 0; i < 4; i++)
                dqt = __builtin_amdgcn_mfma_f64_16x16x4f64(colop(k, kb, i), ds[i], dqt, 0, 0, 0);
        }
        const int s = 16 * j + lr;
        if (s < K)
#pragma unroll
            for (int i = 0; i < 4; i++) dq[base + (int64_t)s * 64 + lk + 4 * i] = scale * dqt[i];
    }
    {
        const int kb = w;
        ConstF64 *tab = exp2_table();
        f64x4 dkt = {0.0, 0.0, 0.0, 0.0}, dvt = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int j = kb; j < nb; j++) {
            asm volatile("" : "+v"(lx));
            f64x4 p, ds;
            grads(tab, j, kb, p, ds);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                Tl[w][0][lr][lk + 4 * i] = p[i];
                Tl[w][1][lr][lk + 4 * i] = ds[i];
            }
            sync();
#pragma unroll
            for (int i = 0; i < 4; i++) {
                dvt = __builtin_amdgcn_mfma_f64_16x16x4f64(colop(dout, j, i), Tl[w][0][4 * i + lk][lr], dvt, 0, 0, 0);
                dkt = __builtin_amdgcn_mfma_f64_16x16x4f64(colop(q, j, i), Tl[w][1][4 * i + lk][lr], dkt, 0, 0, 0);
            }
            sync();  // the tile is rewritten
        }
        const int s = 16 * kb + lr;
        if (s < K)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                dk[base + (int64_t)s * 64 + lk + 4 * i] = scale * dkt[i];
                dv[base + (int64_t)s * 64 + lk + 4 * i] = dvt[i];
            }
    }
}

static unsigned blocks_for(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

bool f64_shape_ok(const nnqs_model_desc &m) { return m.d_model == 64 && m.n_heads == 4 && m.d_ff % 64 == 0; }

nnqs_status f64_model_pack(nnqs_model *m, hipStream_t st) {
    if (!f64_shape_ok(m->desc)) return NNQS_OK;
    if (!m->d_w64p && hipMalloc(&m->d_w64p, f64_packed_bytes(m->desc)) != hipSuccess)
        return fail(NNQS_ENOMEM, "device allocation of the packed model failed");
    f64_pack(model_view(m), m->d_w64p, st);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

// Phase MLP of n configurations (keys, or keys[list]) in passes of kF64Batch.
static nnqs_status enqueue_phase_f64(nnqs_model *m, const uint64_t *keys, const int32_t *list, int64_t n, double *phase,
                                     hipStream_t st) {
    const ModelView M = model_view(m);
    const int P = M.P;
    const int64_t Bmax = n < kF64Batch ? n : kF64Batch;
    const size_t need = (size_t)Bmax * 2 * P * sizeof(double);
    if (m->f64cap < need) {
        NNQS_HIP_CHECK(hipStreamSynchronize(st));
        hipFree(m->d_f64s);
        m->d_f64s = nullptr;
        m->f64cap = 0;
        if (hipMalloc(&m->d_f64s, need) != hipSuccess) return fail(NNQS_ENOMEM, "FP64 forward scratch (%zu bytes)", need);
        m->f64cap = need;
    }
    double *z1 = reinterpret_cast<double *>(m->d_f64s), *z2 = z1 + (size_t)Bmax * P;
    const double *W = m->d_w64;
    for (int64_t b0 = 0; b0 < n; b0 += kF64Batch) {
        const int64_t B = n - b0 < kF64Batch ? n - b0 : kF64Batch;
        const uint64_t *kb = list ? keys : keys + 2 * b0;
        const int32_t *lb = list ? list + b0 : nullptr;
        hipLaunchKernelGGL(k64_phase1, dim3(blocks_for(B * P)), dim3(256), 0, st, M, kb, lb, B, z1);
        gemm64<2, false>(z1, P, W + M.off.ph_w2, P, W + M.off.ph_b2, B, P, P, z2, P, GemmEpi{}, st);
        hipLaunchKernelGGL(k64_phase_out, dim3(blocks_for(B, 4)), dim3(256), 0, st, M, z2, lb, B,
                           list ? phase : phase + b0);
    }
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

nnqs_status enqueue_logpsi_f64(const nnqs_model *cm, const uint64_t *keys, int64_t n, double *logabs,
                               double *phase, hipStream_t st, int cpos, double *cond, double *kvc, double *pre) {
    nnqs_model *m = const_cast<nnqs_model *>(cm);  // owns its scratch (one call at a time per model)
    transformer_f64_sample(model_view(m), m->d_w64p, keys, n, logabs, cpos, cond, kvc, pre, st);
    NNQS_HIP_CHECK(hipGetLastError());
    return phase ? enqueue_phase_f64(m, keys, nullptr, n, phase, st) : NNQS_OK;
}

// FP64 forward of n listed connections (sorted by first changed row block,
// hdr on the device) with prefix reuse from the cache kvc / pre of the
// chunk's samples, indexed by list entry / C.  Results go to xla / xph.
nnqs_status enqueue_f64_list(const nnqs_model *cm, const uint64_t *xkeys, int64_t C, const int32_t *list,
                             const int64_t *hdr, int64_t n, const double *kvc, const double *pre, double *xla,
                             double *xph, hipStream_t st) {
    if (n <= 0) return NNQS_OK;
    nnqs_model *m = const_cast<nnqs_model *>(cm);
    transformer_f64_list(model_view(m), m->d_w64p, xkeys, C, list, hdr, n, kvc, pre, xla, st);
    NNQS_HIP_CHECK(hipGetLastError());
    return enqueue_phase_f64(m, xkeys, list, n, xph, st);
}

// Instances used by the gradient (grad_f64.hip).
template void gemm64<0, true>(const double *, int, const double *, int, const double *, int64_t, int, int, double *, int,
                              const GemmEpi &, hipStream_t);
template void gemm64<3, false>(const double *, int, const double *, int, const double *, int64_t, int, int, double *, int,
                               const GemmEpi &, hipStream_t);
template void gemm64<4, true>(const double *, int, const double *, int, const double *, int64_t, int, int, double *, int,
                              const GemmEpi &, hipStream_t);
template void gemm64<5, false>(const double *, int, const double *, int, const double *, int64_t, int, int, double *, int,
                               const GemmEpi &, hipStream_t);

}  // namespace nnqs
