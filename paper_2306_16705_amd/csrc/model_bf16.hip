// Phase MLP on BF16 MFMA, the BF16 / FP8 copies of the weights, and the
// launches of the reduced-precision network (phase MLP sizes of Section 4.1;
// the transformer's kernel body is in transformer.hpp), for the shape d_model
// 64, 4 heads, FFN 256, phase hidden 512, K <= 64 orbitals.
//
// Phase MLP: bits[128 x 128] @ W1 and GELU(z1)[128 x 512] @ W2 on the 16x16x32
// MFMA for 128 configurations per block, each wave owning 64 output columns
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
// on BF16 MFMA with FP32 accumulation.  A block of kPhWaves waves takes 128
// configurations per pass; wave w owns output columns 64 w .. 64 w + 63 of
// both layers, so each weight fragment is read once per 128 configurations
// (held in registers across the eight groups of 16), the hidden layer z1
// stays in LDS, and the four per-wave partial dot products of each
// configuration are added in wave order at the end.
// In list mode (see TfArgs) the configurations are xkeys[list[k]] for k
// below the total of the four class counts, and phase[list[k]] receives them.
constexpr int kPhWaves = 8, kPhRows = 16 * kPhWaves, kZld = kP + 8;
__global__ void __launch_bounds__(64 * kPhWaves) k_phase_bf16(Bf16View M, TfArgs A, double *__restrict__ phase) {
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
        // z1 = GELU(bits @ W1 + b1) for the block's 128 configurations, this wave's 64 columns;
        // the layer-1 B fragments (W1^T rows col0 + 16 cb + c16) serve all eight groups
        bf16x8 bw1[kPhaseBits / 32][4];
#pragma unroll
        for (int ks = 0; ks < kPhaseBits / 32; ks++)
#pragma unroll
            for (int cb = 0; cb < 4; cb++)
                bw1[ks][cb] =
                    *reinterpret_cast<const bf16x8 *>(w1T + (int64_t)(col0 + cb * 16 + c16) * kPhaseBits + ks * 32 + kq);
        for (int rg = 0; rg < kPhWaves; rg++) {
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
        float part[kPhWaves][4];
#pragma unroll
        for (int rg = 0; rg < kPhWaves; rg++)
#pragma unroll
            for (int i = 0; i < 4; i++) part[rg][i] = 0.f;
#pragma unroll 1
        for (int half = 0; half < 2; half++) {
            f32x4 acc2[kPhWaves][2];
#pragma unroll
            for (int rg = 0; rg < kPhWaves; rg++)
#pragma unroll
                for (int cb = 0; cb < 2; cb++) acc2[rg][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
            for (int ks = 0; ks < kP; ks += 32) {
                bf16x8 bw[2];
#pragma unroll
                for (int cb = 0; cb < 2; cb++)
                    bw[cb] = *reinterpret_cast<const bf16x8 *>(w2T + (int64_t)(col0 + (2 * half + cb) * 16 + c16) * kP +
                                                               ks + kq);
#pragma unroll
                for (int rg = 0; rg < kPhWaves; rg++) {
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
                for (int rg = 0; rg < kPhWaves; rg++)
#pragma unroll
                    for (int i = 0; i < 4; i++) part[rg][i] += gelu32(acc2[rg][cb][i] + bb) * ww;
            }
        }
#pragma unroll
        for (int rg = 0; rg < kPhWaves; rg++) {
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

static uint16_t to_bf16_bits(float f) {  // round to nearest even
    uint32_t u;
    std::memcpy(&u, &f, 4);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// OCP FP8 E4M3 (bias 7, 3 mantissa bits, largest finite 448), round to
// nearest even, saturated at +-448.
static uint8_t to_e4m3(float f) {
    const uint8_t sign = std::signbit(f) ? 0x80 : 0x00;
    double a = std::fabs((double)f);
    if (!(a == a)) return 0x7F;
    if (a >= 448.0) return sign | 0x7E;
    auto rne = [](double v) {  // round half to even
        const double fl = std::floor(v), d = v - fl;
        if (d > 0.5) return fl + 1.0;
        if (d < 0.5) return fl;
        return std::fmod(fl, 2.0) == 0.0 ? fl : fl + 1.0;
    };
    if (a < std::ldexp(1.0, -6)) {  // subnormal: m * 2^-9 (m = 8 carries into the smallest normal)
        return sign | (uint8_t)rne(a * 512.0);
    }
    int e = 0;
    const double fr = std::frexp(a, &e);  // a = fr * 2^e, fr in [0.5, 1)
    e -= 1;                               // a = (2 fr) * 2^e, 2 fr in [1, 2)
    double q = rne((2.0 * fr - 1.0) * 8.0);
    if (q >= 8.0) {
        q = 0.0;
        e += 1;
    }
    const int code = ((e + 7) << 3) | (int)q;
    return sign | (uint8_t)(code > 0x7E ? 0x7E : code);
}

nnqs_status bf16_model_init(nnqs_model *m, const float *weights) {
    const nnqs_model_desc &d = m->desc;
    m->bf16_ok = d.d_model == kD && d.n_heads == kH && d.d_ff == kF && d.phase_hidden == kP && d.n_orb <= 64 &&
                 2 * d.n_orb <= kPhaseBits;
    if (!m->bf16_ok) return NNQS_OK;
    const int K = d.n_orb, L = d.n_layers;
    const ModelOffsets &o = m->off;
    const Bf16Layout bl = bf16_layout(L);
    const F32Layout fl = f32_layout(K, L);
    std::vector<uint16_t> wb((size_t)bl.total, 0);
    std::vector<uint8_t> w8((size_t)bl.total, 0);
    std::vector<float> wf((size_t)fl.total, 0.f);
    auto W = [&](int64_t off) { return weights + off; };
    // transposed copy: dst[n][k] = src[k][n] for a [kdim][ndim] source matrix
    auto put_t = [&](int64_t dst, int dst_ld, const float *src, int kdim, int ndim, int row0) {
        for (int k = 0; k < kdim; k++)
            for (int nn = 0; nn < ndim; nn++) wb[dst + (int64_t)(row0 + nn) * dst_ld + k] = to_bf16_bits(src[k * ndim + nn]);
    };
    // Element (output n, inner k) of a transformer matrix in operand order: 16 x
    // 32 fragments, row block major, lane (k % 32) / 8 * 16 + n % 16 of a
    // fragment holding its eight k one after another.
    auto frag_at = [](int kdim, int n, int k) -> int64_t {
        return ((int64_t)((n >> 4) * (kdim / 32) + (k >> 5)) * 64 + ((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
    };
    // Output n's place among the rows with `pair`: output 32 p + 8 q + 4 t + i
    // in row 4 q + i of block 2 p + t, so that the eight outputs a lane (row
    // group q) holds of two blocks are one operand of the next product.
    auto paired = [](int n) { return (n & ~31) | (n & 4) << 2 | (n & 24) >> 1 | (n & 3); };
    auto put_frag = [&](int64_t dst, const float *src, int kdim, int ndim, int row0, bool pair) {
        for (int k = 0; k < kdim; k++)
            for (int nn = 0; nn < ndim; nn++)
                wb[dst + frag_at(kdim, row0 + (pair ? paired(nn) : nn), k)] = to_bf16_bits(src[k * ndim + nn]);
    };
    // FP8 copy in the same order, with the power of two s that brings the
    // matrix's largest magnitude to at most 448; stores s, 1/s
    auto put_f8 = [&](int64_t dst, const float *src, int kdim, int ndim, int row0, bool pair, float *sc) {
        double mx = 0.0;
        for (int64_t e = 0; e < (int64_t)kdim * ndim; e++) mx = std::max(mx, std::fabs((double)src[e]));
        int k2 = mx > 0.0 ? (int)std::floor(std::log2(448.0 / mx)) : 0;
        k2 = std::min(60, std::max(-60, k2));
        const double s = std::ldexp(1.0, k2);
        for (int k = 0; k < kdim; k++)
            for (int nn = 0; nn < ndim; nn++)
                w8[dst + frag_at(kdim, row0 + (pair ? paired(nn) : nn), k)] = to_e4m3((float)(s * src[k * ndim + nn]));
        sc[0] = (float)s;
        sc[1] = (float)(1.0 / s);
    };
    // A LayerNorm's scale g and shift b fold into the product y W + c that
    // reads it: (n * g + b) W + c = n (diag(g) W) + (b W + c), n = the
    // normalised row; the attention scale 1/sqrt(16) and log2(e) (the softmax
    // runs in base 2) fold into W_q and b_q.  Folded in FP64, then rounded.
    auto fold = [&](const float *Wm, const float *bm, const float *g, const float *beta, int kdim, int ndim,
                    double scale, std::vector<float> &Wf, std::vector<float> &bf) {
        Wf.assign((size_t)kdim * ndim, 0.f);
        bf.assign((size_t)ndim, 0.f);
        for (int nn = 0; nn < ndim; nn++) {
            double acc = bm[nn];
            for (int k = 0; k < kdim; k++) {
                Wf[(size_t)k * ndim + nn] = (float)(scale * (double)g[k] * (double)Wm[(size_t)k * ndim + nn]);
                acc += (double)beta[k] * (double)Wm[(size_t)k * ndim + nn];
            }
            bf[nn] = (float)(scale * acc);
        }
    };
    const double qscale = 0.25 * 1.4426950408889634;
    std::vector<float> fw, fb;
    for (int l = 0; l < L; l++) {
        const int64_t lo = o.layer0 + l * o.layer_stride;
        const int64_t base = bl.layer0 + l * bl.layer_stride;
        const int64_t dd = kD * kD;
        // layer block layout of the FP32 weights: ln1_g ln1_b wq bq wk bk wv bv wo bo ln2_g ln2_b w1 b1 w2 b2
        const float *ln1g = W(lo), *ln1b = W(lo + kD);
        const float *wq = W(lo + 2 * kD), *bq = wq + dd, *wk = bq + kD, *bk = wk + dd, *wv = bk + kD, *bv = wv + dd,
                    *wo = bv + kD, *bo = wo + dd, *ln2g = bo + kD, *ln2b = ln2g + kD, *w1 = ln2b + kD,
                    *b1 = w1 + kD * kF, *w2 = b1 + kF, *b2 = w2 + kF * kD;
        float *lv = wf.data() + fl.layer0 + l * fl.layer_stride;
        fold(wq, bq, ln1g, ln1b, kD, kD, qscale, fw, fb);
        put_frag(base, fw.data(), kD, kD, 0, true);
        put_f8(base, fw.data(), kD, kD, 0, true, lv + kV_f8 + 0);
        std::memcpy(lv + kV_bqkv, fb.data(), kD * 4);
        fold(wk, bk, ln1g, ln1b, kD, kD, 1.0, fw, fb);
        put_frag(base, fw.data(), kD, kD, 64, true);
        put_f8(base, fw.data(), kD, kD, 64, true, lv + kV_f8 + 2);
        std::memcpy(lv + kV_bqkv + 64, fb.data(), kD * 4);
        fold(wv, bv, ln1g, ln1b, kD, kD, 1.0, fw, fb);
        put_frag(base, fw.data(), kD, kD, 128, false);
        put_f8(base, fw.data(), kD, kD, 128, false, lv + kV_f8 + 4);
        std::memcpy(lv + kV_bqkv + 128, fb.data(), kD * 4);
        put_frag(base + 192 * 64, wo, kD, kD, 0, false);
        put_f8(base + 192 * 64, wo, kD, kD, 0, false, lv + kV_f8 + 6);
        fold(w1, b1, ln2g, ln2b, kD, kF, 1.0, fw, fb);
        put_frag(base + 192 * 64 + 64 * 64, fw.data(), kD, kF, 0, true);
        put_f8(base + 192 * 64 + 64 * 64, fw.data(), kD, kF, 0, true, lv + kV_f8 + 8);
        std::memcpy(lv + kV_b1, fb.data(), kF * 4);
        put_frag(base + 192 * 64 + 64 * 64 + 256 * 64, w2, kF, kD, 0, false);
        put_f8(base + 192 * 64 + 64 * 64 + 256 * 64, w2, kF, kD, 0, false, lv + kV_f8 + 10);
        std::memcpy(lv + kV_ln1_g, ln1g, kD * 4);
        std::memcpy(lv + kV_ln1_b, ln1b, kD * 4);
        std::memcpy(lv + kV_bo, bo, kD * 4);
        std::memcpy(lv + kV_ln2_g, ln2g, kD * 4);
        std::memcpy(lv + kV_ln2_b, ln2b, kD * 4);
        std::memcpy(lv + kV_b2, b2, kD * 4);
    }
    std::memcpy(wf.data() + fl.tok_emb, W(o.tok_emb), 5 * kD * 4);
    std::memcpy(wf.data() + fl.pos_emb, W(o.pos_emb), (size_t)K * kD * 4);
    std::memcpy(wf.data() + fl.lnf_g, W(o.lnf_g), kD * 4);
    std::memcpy(wf.data() + fl.lnf_b, W(o.lnf_b), kD * 4);
    fold(W(o.head_w), W(o.head_b), W(o.lnf_g), W(o.lnf_b), kD, 4, 1.0, fw, fb);
    std::memcpy(wf.data() + fl.head_w, fw.data(), 4 * kD * 4);
    std::memcpy(wf.data() + fl.head_b, fb.data(), 4 * 4);
    std::memcpy(wf.data() + fl.bias, W(o.bias), (size_t)4 * K * 4);
    std::memcpy(wf.data() + fl.ph_b1, W(o.ph_b1), kP * 4);
    std::memcpy(wf.data() + fl.ph_b2, W(o.ph_b2), kP * 4);
    std::memcpy(wf.data() + fl.ph_w3, W(o.ph_w3), kP * 4);
    wf[fl.ph_b3] = *W(o.ph_b3);
    for (int i = 0; i < kGeluN; i++) {  // Phi at the knots, in FP64
        const double v0 = (i - (double)kGeluOff) / kGeluScale, v1 = v0 + 1.0 / kGeluScale;
        const double p0 = 0.5 * std::erfc(-v0 / std::sqrt(2.0)), p1 = 0.5 * std::erfc(-v1 / std::sqrt(2.0));
        wf[fl.gelu + 2 * i] = (float)p0;
        wf[fl.gelu + 2 * i + 1] = (float)(p1 - p0);
    }
    // phase W1 [2K][512] -> ph_w1T[512][128] (bits beyond 2K stay zero)
    put_t(bl.ph_w1T, kPhaseBits, W(o.ph_w1), 2 * K, kP, 0);
    put_t(bl.ph_w2T, kP, W(o.ph_w2), kP, kP, 0);
    if (hipMalloc(&m->d_bf16, wb.size() * 2) != hipSuccess || hipMalloc(&m->d_f32, wf.size() * 4) != hipSuccess ||
        hipMalloc(&m->d_fp8, w8.size()) != hipSuccess)
        return fail(NNQS_ENOMEM, "device allocation of the BF16 model failed");
    if (hipMemcpy(m->d_fp8, w8.data(), w8.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(m->d_bf16, wb.data(), wb.size() * 2, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(m->d_f32, wf.data(), wf.size() * 4, hipMemcpyHostToDevice) != hipSuccess)
        return fail(NNQS_EHIP, "copy of the BF16 model failed");
    return NNQS_OK;
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

static unsigned phase_grid(int64_t n) {
    const int64_t cap = (int64_t)cu_count();  // one block per CU (z1 fills most of its LDS)
    const int64_t b = (n + kPhRows - 1) / kPhRows;
    return (unsigned)(b < 1 ? 1 : b < cap ? b : cap);
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
        hipLaunchKernelGGL(k_phase_bf16, dim3(phase_grid(n)), dim3(kPhWaves * 64), 0, st, v, A, phase);
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
        hipLaunchKernelGGL(k_phase_bf16, dim3(phase_grid(max_entries)), dim3(kPhWaves * 64), 0, st, v, A, xph);
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
    hipLaunchKernelGGL(k_phase_bf16, dim3(phase_grid(max_entries)), dim3(kPhWaves * 64), 0, st, bf16_view(m), A, xph);
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
