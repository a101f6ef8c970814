// Kernels of the layer-batched FP64 network forward (model_f64.hip), shared
// with the FP64 backward (grad_f64.hip).
#pragma once

#include "model.hpp"

namespace nnqs {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Previous-token input embeddings h[b*K + s][c] and the token of every row.
__global__ void k64_embed(ModelView M, const uint64_t *__restrict__ keys, int64_t B, int8_t *__restrict__ tok,
                          double *__restrict__ h);
// LayerNorm (eps 1e-5) of rows of width 64, one wave per row.
__global__ void k64_layernorm(const double *__restrict__ in, const double *__restrict__ g,
                              const double *__restrict__ b, int64_t rows, double *__restrict__ out);
// C[r][j] = epi(bias[j] + sum_k A[r][k] B[k][j]); B[k][j] = W[k*ldw + j], or
// W[j*ldw + k] with TB (the transposed weight, y W^T).  EPI 0 stores, 2
// stores GELU, 3 stores GELU' and, in E.C2, GELU (u Phi(u), Phi(u) + u phi(u)),
// 4 stores the sum times E.U, 5 stores E.src + the sum.
struct GemmEpi {
    const double *U = nullptr;    // EPI 4
    const double *src = nullptr;  // EPI 5
    double *C2 = nullptr;         // EPI 3
};

template <int EPI, bool TB>
void gemm64(const double *A, int lda, const double *W, int ldw, const double *bias, int64_t M, int N, int Kd, double *C,
            int ldc, const GemmEpi &E, hipStream_t st);
// C + x cs = a W_x + b_x (x = 0, 1, 2; weights and biases ws apart), and C = sum_x A_x W_x^T.
void gemm64_qkv(const double *a, const double *W, const double *bias, int64_t ws, int64_t M, double *C, int64_t cs,
                hipStream_t st);
void gemm64_qkv_back(const double *A, int64_t as, const double *W, int64_t ws, int64_t M, double *C, hipStream_t st);
// Attention backward of [B*K][64] rows, one block per (configuration, head).
__global__ void k64x_attention_back(const double *__restrict__ q, const double *__restrict__ k,
                                    const double *__restrict__ v, const double *__restrict__ o,
                                    const double *__restrict__ dout, int K, double scale,
                                    double *__restrict__ dq, double *__restrict__ dk, double *__restrict__ dv);
// Causal attention of [B*K][64] rows, one block per (configuration, head).
__global__ void k64_attention(const double *__restrict__ q, const double *__restrict__ k,
                              const double *__restrict__ v, int K, double scale, double *__restrict__ o);
// Output head: log-probability of each row's token.
__global__ void k64_head(ModelView M, const double *__restrict__ a, const int8_t *__restrict__ tok, int64_t B,
                         double *__restrict__ lp);
// log|psi| = 1/2 sum of the rows' log-probabilities; phase = b3 + z2 . w3.
__global__ void k64_finish(ModelView M, const double *__restrict__ lp, const double *__restrict__ z2, int64_t B,
                           double *__restrict__ logabs, double *__restrict__ phase);

// The whole network over n configurations, or over the listed connections
// (chunk-local indices sorted by first row block, hdr = {count[4],
// offset[4]} on the device, n at most in total), in one launch
// (transformer_f64.hip); see enqueue_logpsi_f64 / enqueue_f64_list.  packed:
// f64_packed_bytes of weights in operand order, written by f64_pack.
size_t f64_packed_bytes(const nnqs_model_desc &d);
void f64_pack(const ModelView &M, double *out, hipStream_t st);
void transformer_f64_sample(const ModelView &M, const double *packed, const uint64_t *keys, int64_t n, double *logabs,
                            int cpos, double *cond, double *kvc, double *pre, hipStream_t st);
void transformer_f64_list(const ModelView &M, const double *packed, const uint64_t *xkeys, int64_t C,
                          const int32_t *list, const int64_t *hdr, int64_t n, const double *kvc, const double *pre,
                          double *xla, hipStream_t st);

__device__ __forceinline__ double gelu_f64(double v) { return 0.5 * v * (1.0 + erf(v * 0.70710678118654752440)); }

typedef const __attribute__((address_space(4))) double ConstF64;

static __constant__ const double kExp2F64[12] = {
    1.0, 0.69314718055994529, 0.24022650695910158, 0.055504108664821625,
    0.0096181291075872564, 0.0013333558146406471, 0.00015403530463724353, 1.5252733841556773e-05,
    1.3215432535912375e-06, 1.0178057087733941e-07, 7.0741942972885211e-09, 4.4558179083360645e-10};

// 2^y for y <= 0 (any y whose result is finite), by y = k + r, |r| <= 1/2:
// the degree-11 Chebyshev interpolant of 2^r (relative error 1.1e-16, computed
// in 60 digits) scaled by 2^k.  -infinity gives 0, NaN stays.
// c: exp2_table().
__device__ __forceinline__ ConstF64 *exp2_table() {
    ConstF64 *c = (ConstF64 *)kExp2F64;  // scalar loads, as in gelu_f64_set
    asm volatile("" : "+s"(c));
    return c;
}
__device__ __forceinline__ double exp2_f64(ConstF64 *c, double y) {
    y = y < -1100.0 ? -1100.0 : y;
    const double k = rint(y), r = y - k;
    double p = c[11];
#pragma unroll
    for (int d = 10; d >= 0; d--) p = fma(p, r, c[d]);
    return ldexp(p, (int)k);
}

// GELU of N values at once, branch-free in each (the library erf branches per
// value and holds some sixty constants in registers):
//  |v| < 1 in every lane: v Phi(v) = v/2 + v^2 Q, Q = erf(v/sqrt 2) / (2 v),
//    the degree-10 Chebyshev interpolant in u = 2 v^2 - 1 (rounding error);
//  |v| < 4: the same with degree 24 in u = v^2/8 - 1;
//  4 <= |v| < 8.5, only when a lane holds such a value: v/2 (1 + erf), erf =
//    the degree-26 Chebyshev interpolant in (|v| - 6.25) / 2.25 (7e-17);
//  beyond: erf is +-1 to the last bit.
// Interpolants computed in 60 and 80 digits; against 60 digits on (-4, 4) the
// result errs by 4.8e-16 at most, the library formula by 4.4e-16.
static __constant__ const double kGeluF64[25] = {
    0.17594978076521386, -0.084321449009966548, 0.055934204012194136, -0.036869326349787415,
    0.022518150229022951, -0.012472326944487759, 0.006236960858025279, -0.0028223176494500206,
    0.0011613497941428662, -0.00043702013792020335, 0.00015124504174748659, -4.8397871058261684e-05,
    1.4390494366132986e-05, -3.9936910104193726e-06, 1.038681379628688e-06, -2.540915032134826e-07,
    5.865906821838677e-08, -1.2817650087921307e-08, 2.6584243489263516e-09, -5.2499951184631638e-10,
    9.8786348741347648e-11, -1.7524701401428917e-11, 3.0237531845586125e-12, -5.8734146284930532e-13,
    9.2184657716858799e-14};
static __constant__ const double kGeluNearF64[11] = {
    0.36804899320837464, -0.028676216415723439, 0.0020886272882345942, -0.00012231148823231227,
    5.8843489555905661e-06, -2.390038977460615e-07, 8.3823160788722323e-09, -2.5841505563028942e-10,
    7.1029498607016969e-12, -1.763118123836441e-13, 3.978834938893191e-15};

static __constant__ const double kErfFarF64[27] = {
    0.99999999958954733, 5.9130082067821315e-09, -4.1575838791571674e-08, 1.8989764057644757e-07,
    -6.3252928767372187e-07, 1.6347852124307522e-06, -3.4045703765565249e-06, 5.8542868059968421e-06,
    -8.4440652875108144e-06, 1.031246305665945e-05, -1.0702056976768269e-05, 9.41003243881435e-06,
    -6.9229632004281158e-06, 4.1300843051776234e-06, -1.8375164170226886e-06, 4.2723068885162323e-07,
    1.6679361256563449e-07, -2.5520079718961154e-07, 1.5568750077337869e-07, -5.3648575046441102e-08,
    -1.3781873383946057e-11, 1.4612764936593988e-08, -9.1253057863499008e-09, 1.1879892705783645e-09,
    1.0902330811607256e-09, -4.0270557555620181e-10, 1.374554738893768e-11};

template <int N>
__device__ __forceinline__ void gelu_f64_set(double (&v)[N]) {
    double u[N], r[N];
    bool in1 = true;
#pragma unroll
    for (int k = 0; k < N; k++) in1 = in1 && fabs(v[k]) < 1.0;
    if (__all(in1)) {
        // read by scalar loads at each use: as plain constants they would be held in registers
        ConstF64 *c = (ConstF64 *)kGeluNearF64;
        asm volatile("" : "+s"(c));
#pragma unroll
        for (int k = 0; k < N; k++) {
            u[k] = fma(v[k] * v[k], 2.0, -1.0);
            r[k] = c[10];
        }
#pragma unroll
        for (int d = 9; d >= 0; d--)
#pragma unroll
            for (int k = 0; k < N; k++) r[k] = fma(r[k], u[k], c[d]);
#pragma unroll
        for (int k = 0; k < N; k++) v[k] = fma(v[k] * v[k], r[k], 0.5 * v[k]);
        return;
    }
    ConstF64 *c = (ConstF64 *)kGeluF64;
    asm volatile("" : "+s"(c));
    bool far = false;
#pragma unroll
    for (int k = 0; k < N; k++) {
        far |= fabs(v[k]) >= 4.0;
        u[k] = fma(v[k] * v[k], 0.125, -1.0);
        r[k] = c[24];
    }
#pragma unroll
    for (int d = 23; d >= 0; d--)
#pragma unroll
        for (int k = 0; k < N; k++) r[k] = fma(r[k], u[k], c[d]);
#pragma unroll
    for (int k = 0; k < N; k++) r[k] = fma(v[k] * v[k], r[k], 0.5 * v[k]);
    if (__any(far)) {
        ConstF64 *e = (ConstF64 *)kErfFarF64;
        asm volatile("" : "+s"(e));
#pragma unroll
        for (int k = 0; k < N; k++) {
            const double a = fabs(v[k]), t = (a - 6.25) * (1.0 / 2.25);
            double q = e[26];
#pragma unroll
            for (int d = 25; d >= 0; d--) q = fma(q, t, e[d]);
            q = a >= 8.5 ? 1.0 : q;
            if (a >= 4.0) r[k] = 0.5 * v[k] * (1.0 + copysign(q, v[k]));
        }
    }
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = r[k];
}

}  // namespace nnqs
