// Phase MLP on BF16 MFMA, the BF16 / FP8 copies of the weights, and the
// launches of the reduced-precision network (phase MLP sizes of Section 4.1;
// the transformer's kernel body is in transformer.hpp), for the shape d_model
// 64, 4 heads, FFN 256, phase hidden 512, K <= 64 orbitals.
//
// Phase MLP: bits[128 x 128] @ W1 and GELU(z1)[128 x 512] @ W2 on the 16x16x32
// MFMA for 16 to 128 configurations per block, each wave owning 64 output columns
// (weight fragments from L2, read once per block pass; z1 in LDS).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "transformer.hpp"

namespace nnqs {

static Bf16Layout bf16_layout(int L) {
    Bf16Layout o{};
    o.layer0 = 0;
    o.layer_stride = 192 * 64 + 64 * 64 + 256 * 64 + 64 * 256;
    o.ph_w1T = L * o.layer_stride;
    o.ph_w2T = o.ph_w1T + (int64_t)kP * kPhaseBits;
    o.total = o.ph_w2T + (int64_t)kP * kP;
    return o;
}

static F32Layout f32_layout(int K, int L) {
    F32Layout o{};
    int64_t at = 0;
    o.tok_emb = at; at += 5 * kD;
    o.pos_emb = at; at += (int64_t)K * kD;
    o.layer0 = at;
    o.layer_stride = 2 * kD + 192 + kD + 2 * kD + kF + kD + 12;
    at += L * o.layer_stride;
    o.lnf_g = at; at += kD;
    o.lnf_b = at; at += kD;
    o.head_w = at; at += 4 * kD;
    o.head_b = at; at += 4;
    o.bias = at; at += 4 * (int64_t)K;
    o.ph_b1 = at; at += kP;
    o.ph_b2 = at; at += kP;
    o.ph_w3 = at; at += kP;
    o.ph_b3 = at; at += 1;
    o.gelu = at; at += 2 * kGeluN;
    o.total = at;
    return o;
}

// Phase MLP (Section 4.1): phi = b3 + w3 . GELU(GELU(bits W1 + b1) W2 + b2)
// on BF16 MFMA with FP32 accumulation.  A block of kPhWaves waves takes 16 kGroups
// configurations per pass; wave w owns output columns 64 w .. 64 w + 63 of
// both layers, so each weight fragment is read once per pass (held in
// registers across the groups of 16), the hidden layer z1
// stays in LDS, and the four per-wave partial dot products of each
// configuration are added in wave order at the end.
// In list mode (see TfArgs) the configurations are xkeys[list[k]] for k
// below the total of the four class counts, and phase[list[k]] receives them.
constexpr int kPhWaves = 8, kZld = kP + 8;
template <int kGroups>
__global__ void __launch_bounds__(64 * kPhWaves) k_phase_bf16(Bf16View M, TfArgs A, double *__restrict__ phase) {
    constexpr int kPhRows = 16 * kGroups;
    __shared__ __align__(16) __bf16 zs[kPhRows * kZld];
    __shared__ float parts[kPhWaves][kPhRows];
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c16 = l & 15, r0 = 4 * (l >> 4), kq = 8 * (l >> 4);
    const int col0 = 64 * w;  // this wave's output columns
    const __bf16 *w1T = M.wb + M.bl.ph_w1T, *w2T = M.wb + M.bl.ph_w2T;
    const float *b1 = M.wf + M.fl.ph_b1, *b2 = M.wf + M.fl.ph_b2, *w3 = M.wf + M.fl.ph_w3;
    const int nbits = 2 * M.K;
    const int64_t n = A.list_mode ? A.hdr[0] + A.hdr[1] + A.hdr[2] + A.hdr[3] : A.n;
    for (int64_t base = (int64_t)blockIdx.x * kPhRows; base < n; base += (int64_t)gridDim.x * kPhRows) {
        // z1 = GELU(bits @ W1 + b1) for the block's configurations, this wave's 64 columns;
        // the layer-1 B fragments (W1^T rows col0 + 16 cb + c16) serve all groups
        bf16x8 bw1[kPhaseBits / 32][4];
#pragma unroll
        for (int ks = 0; ks < kPhaseBits / 32; ks++)
#pragma unroll
            for (int cb = 0; cb < 4; cb++)
                bw1[ks][cb] =
                    *reinterpret_cast<const bf16x8 *>(w1T + (int64_t)(col0 + cb * 16 + c16) * kPhaseBits + ks * 32 + kq);
        for (int rg = 0; rg < kGroups; rg++) {
            const int64_t cr = base + 16 * rg + c16;
            Key x{0ull, 0ull};
            if (cr < n) {
                const uint64_t *kp = A.list_mode ? A.xkeys + 2 * (int64_t)A.list[cr] : A.keys + 2 * cr;
                x.lo = kp[0];
                x.hi = kp[1];
            }
            f32x4 acc[4];
#pragma unroll
            for (int cb = 0; cb < 4; cb++) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < kPhaseBits / 32; ks++) {
                bf16x8 ab;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const int p = ks * 32 + kq + e;
                    ab[e] = (__bf16)((p < nbits && key_bit(x, p)) ? 1.0f : 0.0f);
                }
#pragma unroll
                for (int cb = 0; cb < 4; cb++) acc[cb] = mfma16(ab, bw1[ks][cb], acc[cb]);
            }
#pragma unroll
            for (int cb = 0; cb < 4; cb++) {
                const float bb = b1[col0 + cb * 16 + c16];
#pragma unroll
                for (int i = 0; i < 4; i++)
                    zs[(16 * rg + r0 + i) * kZld + col0 + cb * 16 + c16] = (__bf16)gelu32(acc[cb][i] + bb);
            }
        }
        __syncthreads();  // z1 of every column written
        // phi partials: w3 . GELU(z1 @ W2 + b2) over this wave's columns, in two
        // halves of 32 columns (every W2 fragment is still read once per pass)
        float part[kGroups][4];
#pragma unroll
        for (int rg = 0; rg < kGroups; rg++)
#pragma unroll
            for (int i = 0; i < 4; i++) part[rg][i] = 0.f;
#pragma unroll 1
        for (int half = 0; half < 2; half++) {
            f32x4 acc2[kGroups][2];
#pragma unroll
            for (int rg = 0; rg < kGroups; rg++)
#pragma unroll
                for (int cb = 0; cb < 2; cb++) acc2[rg][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll(kGroups == 8 ? 2 : 8)
            for (int ks = 0; ks < kP; ks += 32) {
                bf16x8 bw[2];
#pragma unroll
                for (int cb = 0; cb < 2; cb++)
                    bw[cb] = *reinterpret_cast<const bf16x8 *>(w2T + (int64_t)(col0 + (2 * half + cb) * 16 + c16) * kP +
                                                               ks + kq);
#pragma unroll
                for (int rg = 0; rg < kGroups; rg++) {
                    const bf16x8 a = *reinterpret_cast<const bf16x8 *>(zs + (16 * rg + c16) * kZld + ks + kq);
#pragma unroll
                    for (int cb = 0; cb < 2; cb++) acc2[rg][cb] = mfma16(a, bw[cb], acc2[rg][cb]);
                }
            }
#pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                const int col = col0 + (2 * half + cb) * 16 + c16;
                const float bb = b2[col], ww = w3[col];
#pragma unroll
                for (int rg = 0; rg < kGroups; rg++)
#pragma unroll
                    for (int i = 0; i < 4; i++) part[rg][i] += gelu32(acc2[rg][cb][i] + bb) * ww;
            }
        }
#pragma unroll
        for (int rg = 0; rg < kGroups; rg++) {
#pragma unroll
            for (int i = 0; i < 4; i++) part[rg][i] = dpp_row_sum(part[rg][i]);
            if (c16 == 0)
#pragma unroll
                for (int i = 0; i < 4; i++) parts[w][16 * rg + r0 + i] = part[rg][i];
        }
        __syncthreads();  // every wave's partials written, z1 consumed
        if ((int)threadIdx.x < kPhRows) {
            const int64_t cfg = base + threadIdx.x;
            if (cfg < n) {
                float s = 0.f;
                for (int q = 0; q < kPhWaves; q++) s += parts[q][threadIdx.x];
                phase[A.list_mode ? (int64_t)A.list[cfg] : cfg] = (double)(s + M.wf[M.fl.ph_b3]);
            }
        }
        __syncthreads();  // parts read before the next pass rewrites them
    }
}

static Bf16View bf16_view(const nnqs_model *m) {
    Bf16View v{};
    v.K = m->desc.n_orb;
    v.L = m->desc.n_layers;
    v.n_up = m->desc.n_up;
    v.n_dn = m->desc.n_dn;
    v.wb = reinterpret_cast<const __bf16 *>(m->d_bf16);
    v.w8 = reinterpret_cast<const uint8_t *>(m->d_fp8);
    v.wf = m->d_f32;
    v.bl = bf16_layout(v.L);
    v.fl = f32_layout(v.K, v.L);
    return v;
}

__device__ __forceinline__ uint16_t to_bf16_bits(float f) {  // round to nearest even
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// OCP FP8 E4M3 (bias 7, 3 mantissa bits, largest finite 448), round to
// nearest even, saturated at +-448.
__device__ __forceinline__ uint8_t to_e4m3(float f) {
    const uint8_t sign = (__builtin_bit_cast(uint32_t, f) >> 31) ? 0x80 : 0x00;
    const double a = fabs((double)f);
    if (!(a == a)) return 0x7F;
    if (a >= 448.0) return sign | 0x7E;
    if (a < 0x1p-6)  // subnormal: m * 2^-9 (m = 8 carries into the smallest normal)
        return sign | (uint8_t)rint(a * 512.0);
    int e = ilogb(a);  // a = v * 2^e, v in [1, 2)
    double q = rint((ldexp(a, -e) - 1.0) * 8.0);
    if (q >= 8.0) {
        q = 0.0;
        e += 1;
    }
    const int code = ((e + 7) << 3) | (int)q;
    return sign | (uint8_t)(code > 0x7E ? 0x7E : code);
}

// Element (output n, inner k) of a transformer matrix in operand order: 16 x
// 32 fragments, row block major, lane (k % 32) / 8 * 16 + n % 16 of a
// fragment holding its eight k one after another.
__device__ __forceinline__ int64_t frag_at(int kdim, int n, int k) {
    return ((int64_t)((n >> 4) * (kdim / 32) + (k >> 5)) * 64 + ((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
}

// Output n's place among the rows of a `pair` matrix: output 32 p + 8 q + 4 t
// + i in row 4 q + i of block 2 p + t, so that the eight outputs a lane (row
// group q) holds of two blocks are one operand of the next product.
__device__ __forceinline__ int paired(int n) { return (n & ~31) | (n & 4) << 2 | (n & 24) >> 1 | (n & 3); }

// The BF16, FP8 and FP32 copies of the network from its FP64 weights, rounded
// to FP32 first.  A LayerNorm's scale g and shift b fold into the product
// y W + c that reads it: (n * g + b) W + c = n (diag(g) W) + (b W + c), n = the
// normalised row; the attention scale 1/sqrt(16) and log2(e) (the softmax
// runs in base 2) fold into W_q and b_q.  Folded in FP64 with every product
// and sum rounded (no contraction), then rounded to FP32.  Every FP8 matrix
// is scaled by the power of two that brings its largest magnitude to at most
// 448.  Block: one of a layer's six matrices (its values stay in registers
// between the search for the largest and the two copies), a 64 x 64 tile of a
// phase matrix's transpose, or (last) the head and the vectors.
// The copy is bound by the latency of a block's few loads; done on the host,
// with its two transfers and the reallocation, it took 4.1 ms per optimiser
// step, here 20 us.
constexpr int kRefreshThreads = 1024;
__global__ void __launch_bounds__(kRefreshThreads)
k_bf16_refresh(const double *__restrict__ w64, ModelOffsets o, int K, int L, Bf16Layout bl, F32Layout fl,
               uint16_t *__restrict__ wb, uint8_t *__restrict__ w8, float *__restrict__ wf) {
#pragma clang fp contract(off)
    __shared__ float sh[64][65];
    const int t = threadIdx.x;
    const auto W = [&](int64_t off) { return (float)w64[off]; };
    const auto copy = [&](int64_t dst, int64_t src, int64_t cnt) {
        for (int64_t e = t; e < cnt; e += kRefreshThreads) wf[dst + e] = W(src + e);
    };
    int blk = (int)blockIdx.x;
    if (blk < 6 * L) {
        const int l = blk / 6, x = blk % 6;  // q, k, v, o, w1, w2
        const int64_t dd = kD * kD, bs = dd + kD;  // one square matrix and its bias
        const int64_t ln1 = o.layer0 + l * o.layer_stride, wq = ln1 + 2 * kD, ln2 = wq + 4 * bs, w1 = ln2 + 2 * kD,
                      w2 = w1 + (int64_t)kD * kF + kF;
        const int kdim = x == 5 ? kF : kD, ndim = x == 4 ? kF : kD;
        const int64_t src = x < 4 ? wq + x * bs : x == 4 ? w1 : w2, bias = src + (int64_t)kdim * ndim;
        const int64_t ln = x == 4 ? ln2 : ln1;
        const bool folds = x != 3 && x != 5, pair = x < 2 || x == 4;
        const double scale = x == 0 ? 0.25 * 1.4426950408889634 : 1.0;
        const int64_t dst = bl.layer0 + l * bl.layer_stride +
                            (x < 3 ? x * dd : x == 3 ? 3 * dd : x == 4 ? 4 * dd : 4 * dd + (int64_t)kD * kF);
        const int64_t lv = fl.layer0 + l * fl.layer_stride;
        const int nshift = ndim == kF ? 8 : 6, per = kdim * ndim / kRefreshThreads;  // 4 or 16
        float v[16];
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            if (i >= per) continue;
            const int e = t + i * kRefreshThreads, k = e >> nshift;
            v[i] = W(src + e);
            if (folds) v[i] = (float)(scale * (double)W(ln + k) * (double)v[i]);
            const float av = fabsf(v[i]);
            mx = mx < av ? av : mx;  // a NaN leaves it
        }
        for (int d = 32; d; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
        if ((t & 63) == 0) sh[0][t >> 6] = mx;
        __syncthreads();
        for (int q = 0; q < kRefreshThreads / 64; q++) mx = fmaxf(mx, sh[0][q]);
        int k2 = mx > 0.f ? ilogb(448.0 / (double)mx) : 0;
        k2 = k2 < -60 ? -60 : k2 > 60 ? 60 : k2;
        const double s = ldexp(1.0, k2);
#pragma unroll
        for (int i = 0; i < 16; i++) {
            if (i >= per) continue;
            const int e = t + i * kRefreshThreads, k = e >> nshift, n = e & (ndim - 1);
            const int64_t at = dst + frag_at(kdim, pair ? paired(n) : n, k);
            wb[at] = to_bf16_bits(v[i]);
            w8[at] = to_e4m3((float)(s * (double)v[i]));
        }
        if (t == 0) {
            wf[lv + kV_f8 + 2 * x] = (float)s;
            wf[lv + kV_f8 + 2 * x + 1] = (float)(1.0 / s);
        }
        if (t < ndim) {
            float b = W(bias + t);
            if (folds) {
                double acc = (double)b;
#pragma unroll 8
                for (int k = 0; k < kD; k++) acc += (double)W(ln + kD + k) * (double)W(src + (int64_t)k * ndim + t);
                b = (float)(scale * acc);
            }
            wf[lv + (x < 3 ? kV_bqkv + 64 * x : x == 3 ? kV_bo : x == 4 ? kV_b1 : kV_b2) + t] = b;
        }
        if (x == 3) {
            copy(lv + kV_ln1_g, ln1, 2 * kD);
            copy(lv + kV_ln2_g, ln2, 2 * kD);
        }
        return;
    }
    blk -= 6 * L;
    const int t1 = kP / 64 * (kPhaseBits / 64), t2 = kP / 64 * (kP / 64);
    if (blk < t1 + t2) {  // dst[n][k] = src[k][n]; inputs beyond the 2K bits are zero
        const bool first = blk < t1;
        const int q = first ? blk : blk - t1, kdim = first ? 2 * K : kP, ld = first ? kPhaseBits : kP;
        const int n0 = q % (kP / 64) * 64, k0 = q / (kP / 64) * 64;
        const int64_t src = first ? o.ph_w1 : o.ph_w2, dst = first ? bl.ph_w1T : bl.ph_w2T;
        const int c = t & 63, r = t >> 6;
        for (int i = r; i < 64; i += kRefreshThreads / 64)
            sh[i][c] = k0 + i < kdim ? W(src + (int64_t)(k0 + i) * kP + n0 + c) : 0.f;
        __syncthreads();
        for (int i = r; i < 64; i += kRefreshThreads / 64)
            wb[dst + (int64_t)(n0 + i) * ld + k0 + c] = to_bf16_bits(sh[c][i]);
        return;
    }
    copy(fl.tok_emb, o.tok_emb, 5 * kD);
    copy(fl.pos_emb, o.pos_emb, (int64_t)K * kD);
    copy(fl.lnf_g, o.lnf_g, kD);
    copy(fl.lnf_b, o.lnf_b, kD);
    copy(fl.bias, o.bias, 4 * (int64_t)K);
    copy(fl.ph_b1, o.ph_b1, kP);
    copy(fl.ph_b2, o.ph_b2, kP);
    copy(fl.ph_w3, o.ph_w3, kP);
    copy(fl.ph_b3, o.ph_b3, 1);
    if (t < 4 * kD) wf[fl.head_w + t] = (float)((double)W(o.lnf_g + (t >> 2)) * (double)W(o.head_w + t));
    if (t < 4) {
        double acc = (double)W(o.head_b + t);
#pragma unroll 8
        for (int k = 0; k < kD; k++) acc += (double)W(o.lnf_b + k) * (double)W(o.head_w + 4 * k + t);
        wf[fl.head_b + t] = (float)acc;
    }
}

nnqs_status bf16_model_refresh(nnqs_model *m, hipStream_t st) {
    if (!m->bf16_ok) return NNQS_OK;
    const int K = m->desc.n_orb, L = m->desc.n_layers;
    const unsigned blocks = 6u * (unsigned)L + kP / 64 * (kPhaseBits / 64 + kP / 64) + 1;
    hipLaunchKernelGGL(k_bf16_refresh, dim3(blocks), dim3(kRefreshThreads), 0, st, m->d_w64, m->off, K, L,
                       bf16_layout(L), f32_layout(K, L), reinterpret_cast<uint16_t *>(m->d_bf16),
                       reinterpret_cast<uint8_t *>(m->d_fp8), m->d_f32);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

nnqs_status bf16_model_init(nnqs_model *m) {
    const nnqs_model_desc &d = m->desc;
    m->bf16_ok = d.d_model == kD && d.n_heads == kH && d.d_ff == kF && d.phase_hidden == kP && d.n_orb <= 64 &&
                 2 * d.n_orb <= kPhaseBits;
    if (!m->bf16_ok) return NNQS_OK;
    const Bf16Layout bl = bf16_layout(d.n_layers);
    const F32Layout fl = f32_layout(d.n_orb, d.n_layers);
    if (hipMalloc(&m->d_bf16, (size_t)bl.total * 2) != hipSuccess ||
        hipMalloc(&m->d_f32, (size_t)fl.total * 4) != hipSuccess || hipMalloc(&m->d_fp8, (size_t)bl.total) != hipSuccess)
        return fail(NNQS_ENOMEM, "device allocation of the BF16 model failed");
    std::vector<float> gelu((size_t)2 * kGeluN);
    for (int i = 0; i < kGeluN; i++) {  // Phi at the knots, in FP64
        const double v0 = (i - (double)kGeluOff) / kGeluScale, v1 = v0 + 1.0 / kGeluScale;
        const double p0 = 0.5 * std::erfc(-v0 / std::sqrt(2.0)), p1 = 0.5 * std::erfc(-v1 / std::sqrt(2.0));
        gelu[2 * i] = (float)p0;
        gelu[2 * i + 1] = (float)(p1 - p0);
    }
    if (hipMemcpy(m->d_f32 + fl.gelu, gelu.data(), gelu.size() * 4, hipMemcpyHostToDevice) != hipSuccess)
        return fail(NNQS_EHIP, "copy of the BF16 model failed");
    return bf16_model_refresh(m, nullptr);
}

void bf16_model_free(nnqs_model *m) {
    hipFree(m->d_bf16);
    hipFree(m->d_f32);
    hipFree(m->d_fp8);
    m->d_fp8 = nullptr;
    m->d_bf16 = nullptr;
    m->d_f32 = nullptr;
}

static int cu_count() {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 256;
    return cus;
}

// One block per CU is resident (the weights take 108 KB of LDS); blocks loop
// over tiles, of at least one configuration each.
static unsigned tf_grid(int64_t n) {
    const int64_t cap = cu_count();
    return (unsigned)(n < 1 ? 1 : n < cap ? n : cap);
}

template <int kGroups>
static void phase_launch(int64_t blocks, hipStream_t st, const Bf16View &v, const TfArgs &A, double *phase) {
    hipLaunchKernelGGL(k_phase_bf16<kGroups>, dim3((unsigned)std::max<int64_t>(blocks, 1)), dim3(kPhWaves * 64), 0, st, v,
                       A, phase);
}

// Groups of 16 per block: the fewest that leave at most one block per CU.
// Fewer groups shorten a block's pass (66 configurations in 41 us with eight,
// 24 us with one), more read the weights less often where blocks would follow
// one another (20,011: 41 us with eight, 109 us with one).
static void phase_run(int64_t n, hipStream_t st, const Bf16View &v, const TfArgs &A, double *phase) {
    const int64_t cus = cu_count(), groups = (n + 15) / 16;
    if (groups <= cus) phase_launch<1>(groups, st, v, A, phase);
    else if (groups <= 2 * cus) phase_launch<2>((groups + 1) / 2, st, v, A, phase);
    else if (groups <= 4 * cus) phase_launch<4>((groups + 3) / 4, st, v, A, phase);
    else phase_launch<8>(std::min((groups + 7) / 8, cus), st, v, A, phase);
}

nnqs_status enqueue_logpsi_bf16(const nnqs_model *m, const uint64_t *keys, int64_t n, double *logabs, double *phase,
                                hipStream_t st, bool fp8) {
    if (!m->bf16_ok) return fail(NNQS_EUNSUPPORTED, "BF16 forward needs d_model 64, 4 heads, FFN 256, P 512, K <= 64");
    const Bf16View v = bf16_view(m);
    TfArgs A{};
    A.keys = keys;
    A.n = n;
    A.logabs = logabs;
    if (fp8) {
        TimedRegion tr("k_transformer_fp8", st);
        tf_launch_sample(true, tf_grid(n), st, v, A);
    } else {
        TimedRegion tr("k_transformer_bf16", st);
        tf_launch_sample(false, tf_grid(n), st, v, A);
    }
    {
        TimedRegion tr("k_phase_bf16", st);
        phase_run(n, st, v, A, phase);
    }
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

nnqs_status enqueue_bf16_cond(const nnqs_model *m, const uint64_t *keys, int64_t n, int cpos, double *cond,
                              double *logabs, hipStream_t st) {
    if (!m->bf16_ok) return fail(NNQS_EUNSUPPORTED, "BF16 forward needs d_model 64, 4 heads, FFN 256, P 512, K <= 64");
    TfArgs A{};
    A.keys = keys;
    A.n = n;
    A.logabs = logabs;
    A.cond_pos = cpos;
    A.cond_out = cond;
    TimedRegion tr("k_transformer_bf16", st);
    tf_launch_sample(false, tf_grid(n), st, bf16_view(m), A);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

nnqs_status enqueue_bf16_rows(const nnqs_model *m, const RowsArgs &A, hipStream_t st) {
    if (!m->bf16_ok) return fail(NNQS_EUNSUPPORTED, "BF16 forward needs d_model 64, 4 heads, FFN 256, P 512, K <= 64");
    TimedRegion tr("k_transformer_rows", st);
    return tf_launch_rows(cu_count(), st, bf16_view(m), A);
}

nnqs_status enqueue_phase_bf16(const nnqs_model *m, const uint64_t *keys, int64_t n, double *phase, hipStream_t st) {
    if (!m->bf16_ok) return fail(NNQS_EUNSUPPORTED, "BF16 forward needs d_model 64, 4 heads, FFN 256, P 512, K <= 64");
    TfArgs A{};
    A.keys = keys;
    A.n = n;
    TimedRegion tr("k_phase_bf16", st);
    phase_run(n, st, bf16_view(m), A, phase);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

int64_t bf16_cache_elems(const nnqs_model *m) { return (int64_t)m->desc.n_layers * (kH / 2) * kKvPerPair; }

nnqs_status enqueue_bf16_cached(const nnqs_model *m, const uint64_t *keys, int64_t n, double *logabs, __bf16 *kv,
                                double *pre, hipStream_t st, bool fp8) {
    if (!m->bf16_ok) return fail(NNQS_EUNSUPPORTED, "BF16 forward needs d_model 64, 4 heads, FFN 256, P 512, K <= 64");
    TfArgs A{};
    A.keys = keys;
    A.n = n;
    A.logabs = logabs;
    A.kv_out = kv;
    A.pre_out = pre;
    if (fp8) {
        TimedRegion tr("k_transformer_fp8", st);
        tf_launch_sample(true, tf_grid(n), st, bf16_view(m), A);
    } else {
        TimedRegion tr("k_transformer_bf16", st);
        tf_launch_sample(false, tf_grid(n), st, bf16_view(m), A);
    }
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

nnqs_status enqueue_bf16_list(const nnqs_model *m, const uint64_t *xkeys, int64_t C, const int32_t *list,
                              const int64_t *hdr, int64_t max_entries, const __bf16 *kv, const double *pre,
                              double *xla, double *xph, hipStream_t st, bool fp8) {
    if (!m->bf16_ok) return fail(NNQS_EUNSUPPORTED, "BF16 forward needs d_model 64, 4 heads, FFN 256, P 512, K <= 64");
    const Bf16View v = bf16_view(m);
    TfArgs A{};
    A.kv_in = kv;
    A.pre_in = pre;
    A.list = list;
    A.hdr = hdr;
    A.xkeys = xkeys;
    A.C = C;
    A.xla = xla;
    A.list_mode = 1;  // kv_out / pre_out stay null: list mode only reads the cache
    if (fp8) {
        TimedRegion tr("k_transformer_fp8_list", st);
        tf_launch_list(true, tf_grid(max_entries), st, v, A);
    } else {
        TimedRegion tr("k_transformer_bf16_list", st);
        tf_launch_list(false, tf_grid(max_entries), st, v, A);
    }
    {
        TimedRegion tr("k_phase_bf16", st);
        phase_run(max_entries, st, v, A, xph);
    }
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

size_t bf16_item_bytes() { return sizeof(TfItem); }

int bf16_batch_max_items() { return kMaxTfItems; }

void bf16_list_item(const nnqs_model *m, const uint64_t *xkeys, int64_t C, const int32_t *list, const int64_t *hdr,
                    const __bf16 *kv, const double *pre, double *xla, void *dst) {
    TfItem it{};
    it.M = bf16_view(m);
    it.A.kv_in = kv;
    it.A.pre_in = pre;
    it.A.list = list;
    it.A.hdr = hdr;
    it.A.xkeys = xkeys;
    it.A.C = C;
    it.A.xla = xla;
    it.A.list_mode = 1;
    std::memcpy(dst, &it, sizeof(it));
}

nnqs_status enqueue_bf16_phase_list(const nnqs_model *m, const uint64_t *xkeys, const int32_t *list, const int64_t *hdr,
                                    int64_t max_entries, double *xph, hipStream_t st) {
    TfArgs A{};
    A.list = list;
    A.hdr = hdr;
    A.xkeys = xkeys;
    A.list_mode = 1;
    TimedRegion tr("k_phase_bf16", st);
    phase_run(max_entries, st, bf16_view(m), A, xph);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

nnqs_status enqueue_bf16_batch(const nnqs_model *m0, const void *d_items, int n_items, hipStream_t st) {
    TimedRegion tr("k_transformer_bf16_batch", st);
    tf_launch_batch((unsigned)cu_count(), st, bf16_view(m0), static_cast<const TfItem *>(d_items), n_items);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

}  // namespace nnqs
