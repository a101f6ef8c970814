// FP64 parameter gradients of the ansatz (Section 3.1, Eq. 11 and Fig. 2,
// the Eq. 12 mask, the phase MLP of Section 4.1) and the VMC step around them:
// the gradient estimator of Eq. 7 (Section 2.1), AdamW and the warm-up
// learning rate of Eq. 13 (Section 4.1).
//
// The forward runs layer by layer over passes of kGradBatch configurations,
// keeping every activation the backward needs; the backward walks the layers
// in reverse with row kernels (one wave per row) for the head and LayerNorm,
// one block per (configuration, head) for attention and FP64 MFMA products with
// the transposed weights, and keeps the gradient of every product's output.
// All weight and bias gradients then come from one grouped launch of X^T dY
// products (kg_gemm_tn): its tiles fill the chip where one product's do not.
// Rows are split so that the launch has about two blocks per CU; each split
// writes the gradient's own layout, and one launch adds the splits in a fixed
// order (kg_reduce), so results are reproducible bit for bit.
// 128 configurations at K = 60, one MI355X: the gradient and an
// optimiser step 10.49 ms before (76 weight-gradient launches of a few blocks,
// 4.6 ms; 4.1 ms of host work), 1.08 ms now, of which the grouped products 124 us,
// the 22 layer products 0.45 ms, attention 0.16 ms.
#include <algorithm>
#include <cmath>

#include "f64_kernels.hpp"

namespace nnqs {

constexpr int64_t kGradBatch = 256;  // configurations per pass

// Occupation bits as a [B][N2] matrix of 0 / 1 (the phase MLP's input).
__global__ void kg_bits(const uint64_t *__restrict__ keys, int64_t B, int N2, double *__restrict__ bits) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= B * N2) return;
    const int64_t b = e / N2;
    const int p = (int)(e - b * N2);
    Key x;
    x.lo = keys[2 * b];
    x.hi = keys[2 * b + 1];
    bits[e] = (double)key_bit(x, p);
}

// Output head backward, one wave per row (lane = model column, d = 64).  The
// row's log-probability lp = z_t - log sum_{allowed u} exp z_u enters log|psi|
// with weight 1/2, so with the configuration's cotangent cl:
// dz_u = cl/2 (delta_{u t} - pi_u) over allowed tokens u, 0 for masked ones;
// d(af) = W_head dz.
__global__ void __launch_bounds__(256) kg_head_back(ModelView M, const double *__restrict__ af,
                                                    const int8_t *__restrict__ tok, int64_t B,
                                                    const double *__restrict__ cl, double *__restrict__ dz,
                                                    double *__restrict__ daf) {
    const int K = M.K;
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= B * K) return;  // wave-uniform
    const int64_t b = row / K;
    const int s = (int)(row - b * K);
    const int tr = lane < s ? tok[b * K + lane] : 0;
    const int up = __popcll(__ballot(tr & 1)), dn = __popcll(__ballot(tr >> 1));
    const double *W = M.w64;
    const double av = af[row * 64 + lane];
    double z[4], wc[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
        wc[t] = W[M.off.head_w + lane * 4 + t];
        double v = av * wc[t];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        z[t] = v;
    }
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
    const double coef = 0.5 * cl[b];
    double g[4], acc = 0.0;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        g[t] = ok[t] ? coef * ((t == ts ? 1.0 : 0.0) - exp(z[t] - mx) / den) : 0.0;
        acc += g[t] * wc[t];
    }
    daf[row * 64 + lane] = acc;
    if (lane < 4) dz[row * 4 + lane] = lane == 0 ? g[0] : lane == 1 ? g[1] : lane == 2 ? g[2] : g[3];
}

// LayerNorm backward (eps 1e-5), one wave per row of width 64: with
// xh = (x - mean) r and gy = dy * gamma,
// dx = r (gy - mean(gy) - xh mean(gy xh)); writes dx (+ add) and
// prod = dy * xh (summed over rows for the gain's gradient).  add may alias dx.
__global__ void __launch_bounds__(256) kg_layernorm_back(const double *__restrict__ x, const double *__restrict__ g,
                                                         const double *__restrict__ dy, int64_t rows,
                                                         const double *add, double *dx,
                                                         double *__restrict__ prod) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int64_t e = row * 64 + lane;
    const double v = x[e];
    double s = v;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    const double mean = s / 64.0;
    double q = (v - mean) * (v - mean);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) q += __shfl_xor(q, off, 64);
    const double r = 1.0 / sqrt(q / 64.0 + 1e-5);
    const double xh = (v - mean) * r;
    const double d = dy[e];
    const double gy = d * g[lane];
    double m1 = gy, m2 = gy * xh;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        m1 += __shfl_xor(m1, off, 64);
        m2 += __shfl_xor(m2, off, 64);
    }
    const double out = r * (gy - m1 / 64.0 - xh * (m2 / 64.0));
    dx[e] = (add ? add[e] : 0.0) + out;
    prod[e] = d * xh;
}

// Phase MLP output layer backward: du2[b][i] = cp[b] w3[i] d2[b][i], d2 =
// GELU'(u2).
__global__ void kg_phase_top(const double *__restrict__ d2, const double *__restrict__ w3,
                             const double *__restrict__ cp, int64_t B, int P, double *__restrict__ du2) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= B * P) return;
    const int64_t b = e / P;
    const int j = (int)(e - b * P);
    du2[e] = cp[b] * w3[j] * d2[e];
}

// One weight-gradient product of the grouped launch: out[goff + i N + j] =
// sum over rows r of X[r][i] D[r][j] (i < M, j < N), and out[boff + j] = sum of
// D[r][j] where boff >= 0 (M = 0: only that).
struct TnProblem {
    const double *X, *D;
    int ldx, ldd, M, N;
    int64_t R, goff, boff;
    int tile0, splits;  // first block; row splits of each of its tiles
};
constexpr int kTnMax = 48;  // 3.1 KB of kernel arguments; four layers in one launch
struct TnGroup {
    TnProblem p[kTnMax];
    int n;
};

// Block: one 64 x 64 tile of one product over one split's rows, four waves of
// 16 rows of the tile; rows r in slices of 32 through LDS, the next slice's
// loads in flight.  The blocks of a product's first tile row also add up D's
// columns.  Split z writes part + z total.
__global__ void __launch_bounds__(256) kg_gemm_tn(TnGroup G, int64_t total, double *__restrict__ part) {
    __shared__ double Xs[32][80];
    __shared__ double Ds[32][80];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lr = l & 15, lk = l >> 4;
    int q = 0;
    while (q + 1 < G.n && (int)blockIdx.x >= G.p[q + 1].tile0) q++;
    const TnProblem &P = G.p[q];
    const int b = (int)blockIdx.x - P.tile0, z = b % P.splits, t = b / P.splits;
    const int nt = (P.N + 63) / 64;
    const int i0 = t / nt * 64, j0 = t % nt * 64;
    const int64_t per = (((P.R + P.splits - 1) / P.splits) + 31) & ~(int64_t)31;
    const int64_t rs = z * per, re = rs + per < P.R ? rs + per : P.R;
    const int tc = threadIdx.x & 63, tr = threadIdx.x >> 6;
    const bool xin = i0 + tc < P.M, din = j0 + tc < P.N;
    const double *X = P.X + i0 + tc, *D = P.D + j0 + tc;
    const bool product = P.M > 0, colsum = P.boff >= 0 && i0 == 0;
    double px[8], pd[8], cs = 0.0;
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int64_t r = k0 + tr + 4 * e;
            px[e] = (r < re && xin) ? X[r * P.ldx] : 0.0;
            pd[e] = (r < re && din) ? D[r * P.ldd] : 0.0;
        }
    };
    f64x4 acc[4] = {};
    load(rs);
    for (int64_t k0 = rs; k0 < re; k0 += 32) {
        if (!product) {  // column sums only
#pragma unroll
            for (int e = 0; e < 8; e++) cs += pd[e];
            load(k0 + 32);
            continue;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; e++) {
            Xs[tr + 4 * e][tc] = px[e];
            Ds[tr + 4 * e][tc] = pd[e];
            cs += pd[e];
        }
        __syncthreads();
        load(k0 + 32);
#pragma unroll
        for (int k4 = 0; k4 < 32; k4 += 4) {
            const double a = Xs[k4 + lk][16 * w + lr];
#pragma unroll
            for (int cb = 0; cb < 4; cb++)
                acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Ds[k4 + lk][cb * 16 + lr], acc[cb], 0, 0, 0);
        }
    }
    double *out = part + z * total;
    if (product)
#pragma unroll
        for (int cb = 0; cb < 4; cb++) {
            const int j = j0 + cb * 16 + lr;
            if (j >= P.N) continue;
#pragma unroll
            for (int ii = 0; ii < 4; ii++) {
                const int i = i0 + 16 * w + lk + 4 * ii;
                if (i < P.M) out[P.goff + (int64_t)i * P.N + j] = acc[cb][ii];
            }
        }
    if (colsum) {  // block-uniform: the four row phases of each column in order
        __syncthreads();
        Ds[tr][tc] = cs;
        __syncthreads();
        if (tr == 0 && din) out[P.boff + j0 + tc] = ((Ds[0][tc] + Ds[1][tc]) + Ds[2][tc]) + Ds[3][tc];
    }
}

// Embedding gradients: h0[b, s] = tok_emb[token at s-1] + pos_emb[s].  Block =
// position: the position's sum over b to pos[s], and the sums by input token
// to tokp[s][5] (each of four row phases in order of b, then the phases).
__global__ void __launch_bounds__(256) kg_embed_back(const double *__restrict__ dh, const int8_t *__restrict__ tok,
                                                     int64_t B, int K, double *__restrict__ pos,
                                                     double *__restrict__ tokp) {
    __shared__ double sh[4][6][64];
    const int s = blockIdx.x, c = threadIdx.x & 63, ph = threadIdx.x >> 6;
    double a[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // tokens 0 .. 4, all
    for (int64_t b = ph; b < B; b += 4) {
        const int64_t row = b * K + s;
        const int prev = s == 0 ? 4 : tok[row - 1];
        const double v = dh[row * 64 + c];
        a[5] += v;
#pragma unroll
        for (int t = 0; t < 5; t++) a[t] += t == prev ? v : 0.0;
    }
#pragma unroll
    for (int t = 0; t < 6; t++) sh[ph][t][c] = a[t];
    __syncthreads();
    for (int t = ph; t < 6; t += 4) {
        const double v = ((sh[0][t][c] + sh[1][t][c]) + sh[2][t][c]) + sh[3][t][c];
        if (t == 5) pos[s * 64 + c] = v;
        else tokp[(s * 5 + t) * 64 + c] = v;
    }
}

// grad[e] = (add ? grad[e] : 0) + the splits of part in order: `splits` of the
// transformer's weights (from layer0 up to the logit bias), one of the phase
// MLP's and the position embedding; the token embedding from its K position
// sums; the fixed logit-bias table has none.
__global__ void kg_reduce(ModelOffsets O, int K, const double *__restrict__ part, int splits,
                          const double *__restrict__ tokp, bool add, double *__restrict__ grad) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= O.total) return;
    double s = 0.0;
    if (e >= O.bias && e < O.ph_w1) {
        s = 0.0;
    } else if (e < O.pos_emb) {
        for (int p = 0; p < K; p++) s += tokp[(int64_t)p * 320 + (e - O.tok_emb)];
    } else {
        const int n = e >= O.layer0 && e < O.bias ? splits : 1;
        for (int z = 0; z < n; z++) s += part[(int64_t)z * O.total + e];
    }
    grad[e] = (add ? grad[e] : 0.0) + s;
}

// Eq. 7 cotangents: with p = c / sum c and E = energy[0] + i energy[1],
// cl = 2 p Re(E_loc - E) (for log|psi|), cp = 2 p Im(E_loc - E) (for the phase).
__global__ void kg_vmc_coef(const uint32_t *__restrict__ counts, const double *__restrict__ eloc, int64_t n,
                            const double *__restrict__ energy, double *__restrict__ cl, double *__restrict__ cp) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n) return;
    const double p = (double)counts[b] / energy[2];
    cl[b] = 2.0 * p * (eloc[2 * b] - energy[0]);
    cp[b] = 2.0 * p * (eloc[2 * b + 1] - energy[1]);
}

// AdamW (decoupled weight decay): w <- w (1 - lr wd) - lr mh / (sqrt(vh) + eps)
// with bias-corrected moments; entries in [fix0, fix1) (the fixed logit-bias
// table) are left unchanged with zero moments.
__global__ void kg_adamw(double *__restrict__ w, const double *__restrict__ g, double *__restrict__ m,
                         double *__restrict__ v, int64_t n, int64_t fix0, int64_t fix1, double lr, double b1,
                         double b2, double eps, double wd, double bc1, double bc2) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    if (e >= fix0 && e < fix1) {
        m[e] = 0.0;
        v[e] = 0.0;
        return;
    }
    const double ge = g[e];
    const double me = b1 * m[e] + (1.0 - b1) * ge;
    const double ve = b2 * v[e] + (1.0 - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    const double mh = me / bc1, vh = ve / bc2;
    w[e] = w[e] * (1.0 - lr * wd) - lr * mh / (sqrt(vh) + eps);
}

static unsigned nblocks(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

// Device scratch of one pass (doubles unless noted), carved from one buffer.
// Per layer: the forward's activations (Hin: L + 1; U: GELU' of the hidden
// layer, G: its GELU) and the gradients of the
// products' outputs (dH: L + 1, dH[l] at the input of layer l).
struct GradScratch {
    double *Hin, *A1, *Q, *O, *Hmid, *A2, *U, *G;  // Q: Q, K, V one after another
    double *dH, *dU, *dA2, *prod2, *dHm, *dQ, *dA1, *prod1;
    double *AF, *LP, *bits, *U1, *Z1, *U2, *Z2, *dO, *dAF, *prodf, *dz, *dP1, *dP2, *tokp;
    double *part, *epart, *energy, *cl, *cp;
    int8_t *tok;
};

// Rows per split: K = 60, 128 configurations take 10 splits (1.08 ms a step; 384
// rows the same, 1,536 rows 1.13 ms).
constexpr int64_t kTnSplitRows = 768;

static int tn_splits(int64_t R) { return (int)std::max<int64_t>(1, (R + kTnSplitRows - 1) / kTnSplitRows); }

// Carves the scratch of passes of Bmax configurations (and cotangents of n)
// from `at`; returns the doubles used.
static size_t grad_carve(const nnqs_model *m, int64_t Bmax, int64_t n, double *base, GradScratch &S) {
    const nnqs_model_desc &md = m->desc;
    const size_t K = md.n_orb, d = md.d_model, F = md.d_ff, P = md.phase_hidden, L = md.n_layers;
    const size_t R = (size_t)Bmax * K, B = (size_t)Bmax, Rd = R * d;
    size_t at = 0;
    auto take = [&](size_t cnt) {
        double *p = base ? base + at : nullptr;
        at += (cnt + 3) & ~(size_t)3;  // whole 32-byte loads, as the attention kernels make
        return p;
    };
    S.Hin = take((L + 1) * Rd);
    S.A1 = take(L * Rd);
    S.Q = take(3 * L * Rd);
    S.O = take(L * Rd);
    S.Hmid = take(L * Rd);
    S.A2 = take(L * Rd);
    S.U = take(L * R * F);
    S.G = take(L * R * F);
    S.dH = take((L + 1) * Rd);
    S.dU = take(L * R * F);
    S.dA2 = take(L * Rd);
    S.prod2 = take(L * Rd);
    S.dHm = take(L * Rd);
    S.dQ = take(3 * L * Rd);
    S.dA1 = take(L * Rd);
    S.prod1 = take(L * Rd);
    S.AF = take(Rd);
    S.LP = take(R);
    S.bits = take(B * 2 * K);
    S.U1 = take(B * P);
    S.Z1 = take(B * P);
    S.U2 = take(B * P);
    S.Z2 = take(B * P);
    S.dO = take(Rd);
    S.dAF = take(Rd);
    S.prodf = take(Rd);
    S.dz = take(R * 4);
    S.dP1 = take(B * P);
    S.dP2 = take(B * P);
    S.tokp = take(K * 5 * d);
    S.part = take((size_t)tn_splits((int64_t)R) * (size_t)m->off.total);
    S.epart = take((size_t)kPartialBlocks * 8);
    S.energy = take(8);
    S.cl = take((size_t)n);
    S.cp = take((size_t)n);
    S.tok = reinterpret_cast<int8_t *>(take((R + 7) / 8 + 1));
    return at;
}

static nnqs_status grad_scratch(nnqs_model *m, int64_t n, GradScratch &S, hipStream_t st) {
    const int64_t Bmax = n < kGradBatch ? n : kGradBatch;
    const size_t need = grad_carve(m, Bmax, n, nullptr, S) * sizeof(double);
    if (m->gradcap < need) {
        NNQS_HIP_CHECK(hipStreamSynchronize(st));
        (void)hipFree(m->d_grads);
        m->d_grads = nullptr;
        m->gradcap = 0;
        if (hipMalloc(&m->d_grads, need) != hipSuccess)
            return fail(NNQS_ENOMEM, "FP64 gradient scratch (%zu bytes)", need);
        m->gradcap = need;
    }
    grad_carve(m, Bmax, n, reinterpret_cast<double *>(m->d_grads), S);
    return NNQS_OK;
}

// Collects the products of a pass and launches them in groups.
struct TnLauncher {
    TnGroup G{};
    int blocks = 0;
    int64_t total;
    double *part;
    hipStream_t st;
    void add(const double *X, int ldx, const double *D, int ldd, int64_t R, int M, int N, int64_t goff, int64_t boff,
             int splits) {
        G.p[G.n] = TnProblem{X, D, ldx, ldd, M, N, R, goff, boff, blocks, splits};
        G.n++;
        blocks += splits * std::max(1, (M + 63) / 64) * ((N + 63) / 64);
        if (G.n == kTnMax) flush();
    }
    void flush() {
        if (G.n) hipLaunchKernelGGL(kg_gemm_tn, dim3((unsigned)blocks), dim3(256), 0, st, G, total, part);
        G.n = blocks = 0;
    }
};

bool grad_shape_ok(const nnqs_model_desc &m) { return f64_shape_ok(m) && m.n_orb <= 64; }

// grad = sum_b cl[b] d log|psi_b| / dw + cp[b] d phi_b / dw (device arrays; the
// logit-bias entries stay zero).  With la / ph, the pass's forward values too.
nnqs_status enqueue_model_grad(nnqs_model *m, const uint64_t *keys, int64_t n, const double *cl, const double *cp,
                               double *grad, double *la_out, double *ph_out, hipStream_t st) {
    if (!grad_shape_ok(m->desc))
        return fail(NNQS_EUNSUPPORTED, "gradients need d_model 64, 4 heads, d_ff a multiple of 64 and n_orb <= 64");
    GradScratch S{};
    nnqs_status rc = grad_scratch(m, n, S, st);
    if (rc != NNQS_OK) return rc;
    const ModelView M = model_view(m);
    const int K = M.K, d = M.d, F = M.F, P = M.P, L = M.L;
    const LayerOffsets LO = layer_offsets(d, F);
    const ModelOffsets &OF = m->off;
    double *W = m->d_w64;
    const double scale = 1.0 / sqrt((double)(d / M.H));
    const GemmEpi none{};
    const int64_t Rs = (n < kGradBatch ? n : kGradBatch) * K;  // layer stride in the saved buffers
    for (int64_t b0 = 0; b0 < n; b0 += kGradBatch) {
        const int64_t B = n - b0 < kGradBatch ? n - b0 : kGradBatch;
        const int64_t R = B * K, Rd = R * d;
        auto lay = [&](double *base, int l, int w) { return base + (size_t)l * Rs * w; };
        // ---------------------------------------------------------- forward
        hipLaunchKernelGGL(k64_embed, dim3(nblocks(Rd)), dim3(256), 0, st, M, keys + 2 * b0, B, S.tok, S.Hin);
        for (int l = 0; l < L; l++) {
            const double *Lw = W + OF.layer0 + (int64_t)l * OF.layer_stride;
            double *hin = lay(S.Hin, l, d), *a1 = lay(S.A1, l, d), *q = lay(S.Q, l, 3 * d), *o = lay(S.O, l, d);
            double *hm = lay(S.Hmid, l, d), *a2 = lay(S.A2, l, d), *u = lay(S.U, l, F), *g = lay(S.G, l, F);
            hipLaunchKernelGGL(k64_layernorm, dim3(nblocks(R, 4)), dim3(256), 0, st, hin, Lw + LO.ln1_g, Lw + LO.ln1_b,
                               R, a1);
            gemm64_qkv(a1, Lw + LO.wq, Lw + LO.bq, LO.wk - LO.wq, R, q, Rs * d, st);
            hipLaunchKernelGGL(k64_attention, dim3((unsigned)(4 * B)), dim3(256), 0, st, q, q + Rs * d, q + 2 * Rs * d, K,
                               scale, o);
            GemmEpi res{};
            res.src = hin;
            gemm64<5, false>(o, d, Lw + LO.wo, d, Lw + LO.bo, R, d, d, hm, d, res, st);
            hipLaunchKernelGGL(k64_layernorm, dim3(nblocks(R, 4)), dim3(256), 0, st, hm, Lw + LO.ln2_g, Lw + LO.ln2_b, R,
                               a2);
            GemmEpi both{};
            both.C2 = g;
            gemm64<3, false>(a2, d, Lw + LO.w1, F, Lw + LO.b1, R, F, d, u, F, both, st);
            res.src = hm;
            gemm64<5, false>(g, F, Lw + LO.w2, d, Lw + LO.b2, R, d, F, lay(S.Hin, l + 1, d), d, res, st);
        }
        double *hl = lay(S.Hin, L, d);
        hipLaunchKernelGGL(k64_layernorm, dim3(nblocks(R, 4)), dim3(256), 0, st, hl, W + OF.lnf_g, W + OF.lnf_b, R, S.AF);
        hipLaunchKernelGGL(kg_bits, dim3(nblocks(B * 2 * K)), dim3(256), 0, st, keys + 2 * b0, B, 2 * K, S.bits);
        GemmEpi ph{};
        ph.C2 = S.Z1;
        gemm64<3, false>(S.bits, 2 * K, W + OF.ph_w1, P, W + OF.ph_b1, B, P, 2 * K, S.U1, P, ph, st);
        ph.C2 = S.Z2;
        gemm64<3, false>(S.Z1, P, W + OF.ph_w2, P, W + OF.ph_b2, B, P, P, S.U2, P, ph, st);
        if (la_out && ph_out) {
            hipLaunchKernelGGL(k64_head, dim3(nblocks(R, 4)), dim3(256), 0, st, M, S.AF, S.tok, B, S.LP);
            hipLaunchKernelGGL(k64_finish, dim3(nblocks(B, 4)), dim3(256), 0, st, M, S.LP, S.Z2, B, la_out + b0,
                               ph_out + b0);
        }
        // --------------------------------------------------------- backward
        TnLauncher T{};
        T.total = OF.total;
        T.part = S.part;
        T.st = st;
        const int sp = tn_splits(R);
        hipLaunchKernelGGL(kg_head_back, dim3(nblocks(R, 4)), dim3(256), 0, st, M, S.AF, S.tok, B, cl + b0, S.dz,
                           S.dAF);
        double *dtop = lay(S.dH, L, d);
        hipLaunchKernelGGL(kg_layernorm_back, dim3(nblocks(R, 4)), dim3(256), 0, st, hl, W + OF.lnf_g, S.dAF, R,
                           (const double *)nullptr, dtop, S.prodf);
        T.add(S.AF, d, S.dz, 4, R, d, 4, OF.head_w, OF.head_b, sp);
        T.add(nullptr, 0, S.prodf, d, R, 0, d, 0, OF.lnf_g, sp);
        T.add(nullptr, 0, S.dAF, d, R, 0, d, 0, OF.lnf_b, sp);
        for (int l = L - 1; l >= 0; l--) {
            const double *Lw = W + OF.layer0 + (int64_t)l * OF.layer_stride;
            const int64_t gl = OF.layer0 + (int64_t)l * OF.layer_stride;
            double *a1 = lay(S.A1, l, d), *q = lay(S.Q, l, 3 * d), *o = lay(S.O, l, d), *hm = lay(S.Hmid, l, d);
            double *a2 = lay(S.A2, l, d), *u = lay(S.U, l, F), *g = lay(S.G, l, F);
            double *dout = lay(S.dH, l + 1, d), *dU = lay(S.dU, l, F), *dA2 = lay(S.dA2, l, d), *dHm = lay(S.dHm, l, d);
            double *dQ = lay(S.dQ, l, 3 * d), *dA1 = lay(S.dA1, l, d), *p1 = lay(S.prod1, l, d), *p2 = lay(S.prod2, l, d);
            // feed-forward block: out = hm + GELU(LN2(hm) W1 + b1) W2 + b2
            GemmEpi gb{};
            gb.U = u;
            gemm64<4, true>(dout, d, Lw + LO.w2, d, nullptr, R, F, d, dU, F, gb, st);
            gemm64<0, true>(dU, F, Lw + LO.w1, F, nullptr, R, d, F, dA2, d, none, st);
            hipLaunchKernelGGL(kg_layernorm_back, dim3(nblocks(R, 4)), dim3(256), 0, st, hm, Lw + LO.ln2_g, dA2, R,
                               (const double *)dout, dHm, p2);
            T.add(g, F, dout, d, R, F, d, gl + LO.w2, gl + LO.b2, sp);
            T.add(a2, d, dU, F, R, d, F, gl + LO.w1, gl + LO.b1, sp);
            T.add(nullptr, 0, p2, d, R, 0, d, 0, gl + LO.ln2_g, sp);
            T.add(nullptr, 0, dA2, d, R, 0, d, 0, gl + LO.ln2_b, sp);
            // attention block: hm = h + Attn(LN1(h)) Wo + bo
            gemm64<0, true>(dHm, d, Lw + LO.wo, d, nullptr, R, d, d, S.dO, d, none, st);
            hipLaunchKernelGGL(k64x_attention_back, dim3((unsigned)(4 * B)), dim3(256), 0, st, q, q + Rs * d, q + 2 * Rs * d,
                               o, S.dO, K, scale, dQ, dQ + Rs * d, dQ + 2 * Rs * d);
            gemm64_qkv_back(dQ, Rs * d, Lw + LO.wq, LO.wk - LO.wq, R, dA1, st);
            hipLaunchKernelGGL(kg_layernorm_back, dim3(nblocks(R, 4)), dim3(256), 0, st, lay(S.Hin, l, d),
                               Lw + LO.ln1_g, dA1, R, (const double *)dHm, lay(S.dH, l, d), p1);
            T.add(o, d, dHm, d, R, d, d, gl + LO.wo, gl + LO.bo, sp);
            T.add(a1, d, dQ, d, R, d, d, gl + LO.wq, gl + LO.bq, sp);
            T.add(a1, d, dQ + Rs * d, d, R, d, d, gl + LO.wk, gl + LO.bk, sp);
            T.add(a1, d, dQ + 2 * Rs * d, d, R, d, d, gl + LO.wv, gl + LO.bv, sp);
            T.add(nullptr, 0, p1, d, R, 0, d, 0, gl + LO.ln1_g, sp);
            T.add(nullptr, 0, dA1, d, R, 0, d, 0, gl + LO.ln1_b, sp);
        }
        hipLaunchKernelGGL(kg_embed_back, dim3((unsigned)K), dim3(256), 0, st, S.dH, S.tok, B, K, S.part + OF.pos_emb,
                           S.tokp);
        // phase MLP: phi = b3 + GELU(GELU(bits W1 + b1) W2 + b2) w3
        hipLaunchKernelGGL(kg_phase_top, dim3(nblocks(B * P)), dim3(256), 0, st, S.U2, W + OF.ph_w3, cp + b0, B, P,
                           S.dP2);
        GemmEpi gb{};
        gb.U = S.U1;
        gemm64<4, true>(S.dP2, P, W + OF.ph_w2, P, nullptr, B, P, P, S.dP1, P, gb, st);
        T.add(S.Z1, P, S.dP2, P, B, P, P, OF.ph_w2, OF.ph_b2, 1);
        T.add(S.bits, 2 * K, S.dP1, P, B, 2 * K, P, OF.ph_w1, OF.ph_b1, 1);
        T.add(S.Z2, P, cp + b0, 1, B, P, 1, OF.ph_w3, OF.ph_b3, 1);
        T.flush();
        hipLaunchKernelGGL(kg_reduce, dim3(nblocks(OF.total)), dim3(256), 0, st, OF, K, (const double *)S.part, sp,
                           (const double *)S.tokp, b0 > 0, grad);
        NNQS_HIP_CHECK(hipGetLastError());
    }
    return NNQS_OK;
}

}  // namespace nnqs

using namespace nnqs;

extern "C" {

nnqs_status nnqs_model_grad(nnqs_model *m, const uint64_t *keys, int64_t n, const double *c_logabs,
                            const double *c_phase, double *grad, double *logabs, double *phase, void *stream) {
    clear_error();
    if (!m || !keys || !c_logabs || !c_phase || !grad) return fail(NNQS_EINVAL, "null pointer argument");
    if (n <= 0) return fail(NNQS_EINVAL, "n must be positive");
    if ((logabs == nullptr) != (phase == nullptr)) return fail(NNQS_EINVAL, "logabs and phase go together");
    return enqueue_model_grad(m, keys, n, c_logabs, c_phase, grad, logabs, phase, as_stream(stream));
}

nnqs_status nnqs_vmc_gradient(nnqs_model *m, const uint64_t *keys, const uint32_t *counts, const double *eloc,
                              int64_t n, double *grad, double *energy, void *stream) {
    clear_error();
    if (!m || !keys || !counts || !eloc || !grad) return fail(NNQS_EINVAL, "null pointer argument");
    if (n <= 0) return fail(NNQS_EINVAL, "n must be positive");
    if (!grad_shape_ok(m->desc))
        return fail(NNQS_EUNSUPPORTED, "gradients need d_model 64, 4 heads, d_ff a multiple of 64 and n_orb <= 64");
    hipStream_t st = as_stream(stream);
    GradScratch S{};
    nnqs_status rc = grad_scratch(m, n, S, st);
    if (rc != NNQS_OK) return rc;
    double *E = energy ? energy : S.energy;
    rc = enqueue_energy_partials(S.epart, counts, eloc, n, E, st);
    if (rc != NNQS_OK) return rc;
    hipLaunchKernelGGL(kg_vmc_coef, dim3(nblocks(n)), dim3(256), 0, st, counts, eloc, n, E, S.cl, S.cp);
    NNQS_HIP_CHECK(hipGetLastError());
    return enqueue_model_grad(m, keys, n, S.cl, S.cp, grad, nullptr, nullptr, st);
}

double nnqs_lr_schedule(int64_t step, int32_t d_model, int32_t warmup) {
    if (step < 1 || d_model < 1 || warmup < 1) return 0.0;
    const double i = (double)step;
    const double a = 1.0 / std::sqrt(i), b = i * std::pow((double)warmup, -1.5);
    return (a < b ? a : b) / std::sqrt((double)d_model);
}

nnqs_status nnqs_model_adamw_step(nnqs_model *m, const double *grad, int64_t step, double lr, double beta1,
                                  double beta2, double eps, double weight_decay, double *mom1, double *mom2,
                                  void *stream) {
    clear_error();
    if (!m || !grad || !mom1 || !mom2) return fail(NNQS_EINVAL, "null pointer argument");
    if (step < 1) return fail(NNQS_EINVAL, "step counts from 1");
    if (!(beta1 >= 0.0 && beta1 < 1.0 && beta2 >= 0.0 && beta2 < 1.0 && eps > 0.0 && lr >= 0.0 &&
          weight_decay >= 0.0))
        return fail(NNQS_EINVAL, "AdamW hyper-parameters out of range");
    hipStream_t st = as_stream(stream);
    const int64_t nw = m->off.total;
    const double bc1 = 1.0 - std::pow(beta1, (double)step), bc2 = 1.0 - std::pow(beta2, (double)step);
    // the weights change in place: no stream may still be reading the old ones
    NNQS_HIP_CHECK(hipDeviceSynchronize());
    hipLaunchKernelGGL(kg_adamw, dim3(nblocks(nw)), dim3(256), 0, st, m->d_w64, grad, mom1, mom2, nw, m->off.bias,
                       m->off.bias + 4 * (int64_t)m->desc.n_orb, lr, beta1, beta2, eps, weight_decay, bc1, bc2);
    NNQS_HIP_CHECK(hipGetLastError());
    // the packed and reduced-precision copies follow the FP64 master weights
    nnqs_status rc = f64_model_pack(m, st);
    if (rc == NNQS_OK) rc = bf16_model_refresh(m, st);
    if (rc != NNQS_OK) return rc;
    NNQS_HIP_CHECK(hipStreamSynchronize(st));  // the new weights hold for every stream once this returns
    return NNQS_OK;
}

nnqs_status nnqs_model_get_weights(const nnqs_model *m, double *out, void *stream) {
    clear_error();
    if (!m || !out) return fail(NNQS_EINVAL, "null pointer argument");
    hipStream_t st = as_stream(stream);
    NNQS_HIP_CHECK(hipMemcpyAsync(out, m->d_w64, m->off.total * sizeof(double), hipMemcpyDeviceToDevice, st));
    return NNQS_OK;
}

}  // extern "C"
