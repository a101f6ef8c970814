// BF16 / FP8 MFMA forward of the amplitude transformer (the network of
// Section 3.1 / Fig. 2) for d_model 64, 4 heads, FFN 256, K <= 64 orbitals:
// device layouts, MFMA operands and the kernel body, instantiated by
// transformer_*.hip.  Every matrix product runs on the 16x16x32 MFMA with
// FP32 accumulation; LayerNorm, softmax, GELU and the output head stay FP32.
#pragma once

#include <algorithm>
#include <cmath>

#include "model.hpp"

namespace nnqs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 64, kH = 4, kDh = 16, kF = 256, kP = 512;
constexpr int kPhaseBits = 128;

// Device layout of the BF16 weights (element offsets into d_bf16).
struct Bf16Layout {
    // per layer: wqkvT[192][64] woT[64][64] w1T[256][64] w2T[64][256], each as
    // 16-row x 32-column operand fragments (see frag_at)
    int64_t layer0, layer_stride;
    int64_t ph_w1T, ph_w2T, total;  // ph_w1T[512][128] (rows: hidden unit, cols: bit), ph_w2T[512][512]
};
// FP32 vectors (element offsets into d_f32).
struct F32Layout {
    int64_t tok_emb, pos_emb, layer0, layer_stride;  // per layer: ln1_g ln1_b bqkv[192] bo ln2_g ln2_b b1[256] b2
    int64_t lnf_g, lnf_b, head_w, head_b, bias, ph_b1, ph_b2, ph_w3, ph_b3, gelu, total;
};

// The transformer's FFN GELU, v * Phi(v), takes the normal CDF Phi from a
// table of kGeluN (value, step) pairs at spacing 1/kGeluScale on [-8, 8):
// linear interpolation errs by at most h^2/8 max|Phi''| = 3e-5 (h = 1/32),
// well below the BF16 rounding of the result; Phi is clamped to its end
// values outside the range (Phi(-8) = 6e-16).  It replaces the exp and
// reciprocal of a closed-form erf by one LDS read (16384 GELUs per layer and
// configuration make this the largest VALU cost of the forward).
constexpr int kGeluN = 512;
constexpr float kGeluScale = 32.0f, kGeluOff = 256.0f, kGeluMaxU = 511.99997f;

// per-layer FP32 vector offsets
constexpr int kV_ln1_g = 0, kV_ln1_b = 64, kV_bqkv = 128, kV_bo = 320, kV_ln2_g = 384, kV_ln2_b = 448,
              kV_b1 = 512, kV_b2 = 768;
// FP8 scales of one layer's six weight matrices (q, k, v, o, w1, w2): for
// each, the power of two s applied before quantisation and 1/s.
constexpr int kV_f8 = 832;

struct Bf16View {
    int K, L, n_up, n_dn;
    const __bf16 *wb;
    const uint8_t *w8;  // FP8 E4M3 copy of the transformer matrices, same element layout as wb
    const float *wf;
    Bf16Layout bl;
    F32Layout fl;
};

// ------------------------------------------------------------ fragments
// v_mfma_f32_16x16x32_bf16 operand layout: A/B lane l holds row/column
// (l & 15) and k = 8 (l >> 4) .. 8 (l >> 4) + 7; the accumulator lane l holds
// column (l & 15) and rows 4 (l >> 4) .. 4 (l >> 4) + 3.
__device__ __forceinline__ f32x4 mfma16(const bf16x8 &a, const bf16x8 &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float dpp_row_sum(float v) {
    // sum over the 16 lanes of a DPP row (all lanes receive the total)
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));  // xor 1
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));  // xor 2
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true)); // half mirror
    v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true)); // mirror
    return v;
}

__device__ __forceinline__ float gelu32(float v) { return gelu_bf16path(v); }

// GELU from the LDS table (see kGeluN): u = 32 (v + 8) clamped to [0, 512),
// entry floor(u), fraction u - floor(u).
__device__ __forceinline__ float gelu_tab(const float2 *tab, float v) {
    const float u = __builtin_amdgcn_fmed3f(fmaf(v, kGeluScale, kGeluOff), 0.0f, kGeluMaxU);
    const float2 e = tab[(int)u];
    return v * fmaf(__builtin_amdgcn_fractf(u), e.y, e.x);
}

// Operands of the four weight products (QKV, output, FFN in and out):
// BF16 on v_mfma_f32_16x16x32_bf16, or OCP FP8 E4M3 bytes on
// v_mfma_f32_16x16x32_fp8_fp8 (same lane layout, eight 1-byte elements per
// lane; activations are not scaled, each weight matrix has a power-of-two
// scale that the accumulators undo).
template <bool kF8>
struct Op;

template <>
struct Op<false> {
    typedef __bf16 T;
    typedef bf16x8 Frag;
    static __device__ __forceinline__ f32x4 mma(const Frag &a, const Frag &b, const f32x4 &c) { return mfma16(a, b, c); }
};

template <>
struct Op<true> {
    typedef uint8_t T;
    typedef long Frag;
    static __device__ __forceinline__ f32x4 mma(const Frag &a, const Frag &b, const f32x4 &c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, c, 0, 0, 0);
    }
};

__device__ __forceinline__ uint32_t fp8x4(const f32x4 &v) {
    int r = 0;
    r = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(v[0], -448.f, 448.f),
                                        __builtin_amdgcn_fmed3f(v[1], -448.f, 448.f), r, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(v[2], -448.f, 448.f),
                                        __builtin_amdgcn_fmed3f(v[3], -448.f, 448.f), r, true);
    return (uint32_t)r;
}

// ------------------------------------------------------ transformer forward
// Work of one launch, in one of two modes.
//  * Sample mode: configurations keys[0..n), every row evaluated; log|psi|
//    to logabs[i].  With `kv_out` and `pre_out` it also keeps, per configuration,
//    every layer's keys and values (BF16, as the attention used them) and the
//    prefix sums pre[i][b] of its per-position log-probabilities over the
//    first 16 b positions: the cache that list mode reads.
//  * List mode: connected configurations x' of cached samples, as chunk-local
//    connection indices e (key xkeys[e], sample e / C) sorted into four
//    classes (hdr = {count[4], offset[4]} on the device).  Class b holds the
//    x' whose first position that differs from their sample lies at or after
//    16 b: by causality the rows s <= 16 b of x' equal the sample's, so only
//    row blocks from b on are evaluated; their attention reads the keys and values
//    of blocks < b from the sample's cache, and the log-probabilities of
//    positions < 16 b are the sample's prefix sum.  log|psi| goes to xla[e].
//    Results are bit-identical to sample mode on x' (same per-row arithmetic,
//    same summation order).
struct TfArgs {
    const uint64_t *keys;
    int64_t n;
    double *logabs;
    __bf16 *kv_out;        // sample mode: cache written (may be null)
    double *pre_out;
    const __bf16 *kv_in;   // list mode: cache read
    const double *pre_in;
    const int32_t *list;
    const int64_t *hdr;
    const uint64_t *xkeys;
    int64_t C;
    double *xla;
    int list_mode;
    int cond_pos;      // sample mode, batch sampling: position whose conditionals are written
    double *cond_out;  // [n][4] masked log-probabilities of the four tokens there (may be null)
};

// One item of a batched list-mode launch: a system's model and work.
struct TfItem {
    Bf16View M;
    TfArgs A;
};
constexpr int kMaxTfItems = 64;
constexpr int kKvPerPair = 64 * 2 * kDh + 2 * kDh * 64;  // cached K [64][32] then V^T [32][64] of a pair of heads

// A wave owns whole configurations: the NB row blocks (16 rows each) of CPW
// configurations, CPW = 4 / NB (one for NB = 3), so up to 64 rows, and
// everything a row passes between products stays in the wave's registers.
// The residual stream and every product's output are kept transposed: lane l
// holds row (l & 15) of a block and, of tile t, columns 16 t + 4 (l >> 4) + i,
// i = 0..3.  The next product wants its B operand as columns 8 (l >> 4) .. + 7
// of a run of 32.  Where the product's rows can be dealt out freely (Q, K,
// FFN hidden units) the weights' rows are stored in the order that gives each
// lane those eight columns from two tiles (`both`); elsewhere `join` makes
// them with two v_permlane32_swap and two v_permlane16_swap.  Q and K carry
// two heads at once, one in the lanes < 32 and one in the others, and the
// other head's lanes of Q are cleared for each score product.  V is produced
// untransposed, which is the A operand of V^T P^T.  LDS then holds only what
// all waves share, the weights in operand order (1 KB, or 512 B in FP8, per
// 16 x 32 fragment: conflict-free reads of lane x 16 bytes), in two halves,
// attention and FFN, so that one is loaded (global_load_lds) while the other
// is in use: two barriers per layer.
//
// Bound: VALU issue (softmax, GELU, LayerNorm, conversions: about 1,200
// instructions per row block and layer beside 118 MFMAs; VALU active 68 % of
// the cycles, MFMA 20 %).  Three waves per SIMD instead of two gain nothing
// (12 waves per block: 1,265 against 1,146 us below).  Against rows staged
// through LDS, two row blocks per wave and 19 barriers per layer (one
// MI355X, whole calls): log|psi| of 20,011 configurations at K = 60 1,618 ->
// 1,077 us; E_loc of 65 samples at K = 24 (1.07e6 x', whose two row blocks
// the earlier tiles padded to four) 87.4 -> 27.3 ms.
constexpr int kTfWaves = 8;

struct Quad2 {
    uint32_t w[2];
};

template <bool kF8>
struct Act;
template <>
struct Act<false> {  // four BF16 of a tile: two words
    typedef Quad2 Q;
    static __device__ __forceinline__ Q pack(const f32x4 &v) {
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = (__bf16)v[i];
        return __builtin_bit_cast(Q, o);
    }
};
template <>
struct Act<true> {  // four FP8 of a tile: one word
    typedef uint32_t Q;
    static __device__ __forceinline__ Q pack(const f32x4 &v) { return fp8x4(v); }
};

// (a, b) -> (a's even row groups of the lower half, ...): lane group q of the
// pair ends with elements 8 q .. 8 q + 3 of [a | b] in a and 8 q + 4 .. + 7 in b
__device__ __forceinline__ void join_word(uint32_t &a, uint32_t &b) {
    const auto h = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    const auto r = __builtin_amdgcn_permlane16_swap(h[0], h[1], false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ bf16x8 both(Quad2 a, Quad2 b) {
    return __builtin_bit_cast(bf16x8, make_uint4(a.w[0], a.w[1], b.w[0], b.w[1]));
}
__device__ __forceinline__ long both(uint32_t a, uint32_t b) { return (long)(((uint64_t)b << 32) | a); }
__device__ __forceinline__ bf16x8 half(const bf16x8 v, uint32_t mask) {  // mask: all ones in the lanes kept, else 0
    const uint4 u = __builtin_bit_cast(uint4, v);
    return __builtin_bit_cast(bf16x8, make_uint4(u.x & mask, u.y & mask, u.z & mask, u.w & mask));
}
__device__ __forceinline__ bf16x8 join(Quad2 a, Quad2 b) {
    join_word(a.w[0], b.w[0]);
    join_word(a.w[1], b.w[1]);
    return both(a, b);
}
__device__ __forceinline__ long join(uint32_t a, uint32_t b) {
    join_word(a, b);
    return both(a, b);
}

// v and v of the lane group 16 (32) lanes away, in either order (the words
// go through scalars: a bit cast of a vector element itself reads element 0).
struct FPair {
    float a, b;
};
__device__ __forceinline__ FPair swap_x16(float v) {
    const uint32_t x = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const uint32_t a = r[0], b = r[1];
    return {__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ __forceinline__ FPair swap_x32(float v) {
    const uint32_t x = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const uint32_t a = r[0], b = r[1];
    return {__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ __forceinline__ float sum_groups(float v) {  // over the four lanes l, l ^ 16, l ^ 32, l ^ 48
    const FPair p = swap_x16(v);
    const FPair q = swap_x32(p.a + p.b);
    return q.a + q.b;
}
__device__ __forceinline__ float max_groups(float v) {
    const FPair p = swap_x16(v);
    const FPair q = swap_x32(fmaxf(p.a, p.b));
    return fmaxf(q.a, q.b);
}

__device__ __forceinline__ f32x4 ld4(const float *p) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    return f32x4{v.x, v.y, v.z, v.w};
}

// Mean and 1/sqrt(var + eps) of a row (four lanes l, l ^ 16, l ^ 32, l ^ 48),
// one-pass statistics.
__device__ __forceinline__ void row_stats(const f32x4 (&h)[4], float &rstd, float &shift) {
    float s = 0.f, s2 = 0.f;
#pragma unroll
    for (int db = 0; db < 4; db++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float v = h[db][i];
            s += v;
            s2 = fmaf(v, v, s2);
        }
    s = sum_groups(s);
    s2 = sum_groups(s2);
    const float mean = s * (1.0f / kD);
    const float var = fmaxf(s2 * (1.0f / kD) - mean * mean, 0.0f);
    rstd = __builtin_amdgcn_rsqf(var + 1e-5f);  // the argument is never subnormal
    shift = -mean * rstd;
}

// The normalised row as B operands of the next product (k = 0..31, 32..63);
// the LayerNorm's scale and shift are folded into that product's weights.
template <bool kF8>
__device__ __forceinline__ void normalize(const f32x4 (&h)[4], typename Op<kF8>::Frag (&x)[2]) {
    float rstd, sh;
    row_stats(h, rstd, sh);
    typename Act<kF8>::Q p[4];
#pragma unroll
    for (int db = 0; db < 4; db++) {
        f32x4 y;
#pragma unroll
        for (int i = 0; i < 4; i++) y[i] = fmaf(h[db][i], rstd, sh);
        p[db] = Act<kF8>::pack(y);
    }
    x[0] = join(p[0], p[1]);
    x[1] = join(p[2], p[3]);
}

// Shared memory of a block: the two weight halves of a layer in operand
// order, the layer's FP32 vectors (two layers in turn), the GELU table.
constexpr int kAttnElems = 192 * 64 + 64 * 64, kFfnElems = 2 * 256 * 64;
constexpr int kVecFloats = 1024;  // one layer's vectors (844 floats) and what follows them
template <bool kF8>
struct TfLds {
    typename Op<kF8>::T wa[kAttnElems];
    typename Op<kF8>::T wf[kFfnElems];
    float vec[2][kVecFloats];
    float2 gtab[kGeluN];
};

// 64 lanes x 16 bytes from src to the wave-uniform LDS address dst.
__device__ __forceinline__ void lds_load_1k(const void *src, void *dst) {
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void *)(reinterpret_cast<const uint8_t *>(src) + 16 * (threadIdx.x & 63)),
        (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// Loads one half of a layer's weights; pieces of 1 KB dealt to the waves in
// turn.  Every wave waits for its own pieces before the barrier that hands
// them over (weights_ready).
template <typename T>
__device__ __forceinline__ void load_half(T *dst, const T *src, int elems, int w) {
    const int pieces = elems * (int)sizeof(T) / 1024;
    for (int p = w; p < pieces; p += kTfWaves)
        lds_load_1k(reinterpret_cast<const uint8_t *>(src) + 1024 * p, reinterpret_cast<uint8_t *>(dst) + 1024 * p);
}

__device__ __forceinline__ void weights_ready() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

template <bool kF8>
__device__ __forceinline__ typename Op<kF8>::Frag wfrag(const typename Op<kF8>::T *base, int f) {
    return *reinterpret_cast<const typename Op<kF8>::Frag *>(base + (f * 64 + (threadIdx.x & 63)) * 8);
}

// Causal attention of one configuration's row block QB for one head:
// S^T[key][query] = K Q^T (the lane owns query l & 15 of the block and keys
// 16 kb + 4 (l >> 4) + i), softmax over keys in base 2 (scale and log2(e) are
// folded into Q), unnormalised weights in BF16, then O^T = V^T P^T divided by
// the row sums 1^T P^T of the same BF16 weights (the same MFMA with an
// all-ones operand).  kf: K operands of blocks 0 .. QB; vf: V^T operands of
// the block pairs (0, 1), (2, 3).  QB is a constant at every call.
__device__ __forceinline__ f32x4 attend(const int QB, const bf16x8 qf, const bf16x8 (&kf)[4], const bf16x8 (&vf)[2]) {
    const int l = threadIdx.x & 63;
    const int c16 = l & 15, r0 = 4 * (l >> 4);
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; e++) ones[e] = (__bf16)1.0f;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 st[4];
#pragma unroll
    for (int kb = 0; kb < 4; kb++)
        if (kb <= QB) st[kb] = mfma16(kf[kb], qf, zero);
    // key 16 kb + r0 + i is visible to query 16 QB + c16 when kb < QB, or
    // kb == QB and r0 + i <= c16
#pragma unroll
    for (int i = 0; i < 4; i++) st[QB][i] = r0 + i <= c16 ? st[QB][i] : -INFINITY;
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 4; kb++)
        if (kb <= QB)
#pragma unroll
            for (int i = 0; i < 4; i++) mx = __builtin_amdgcn_fmed3f(mx, st[kb][i], INFINITY);  // the larger
    mx = max_groups(mx);
    Quad2 pq[4];
#pragma unroll
    for (int kb = 0; kb < 4; kb++) {
        pq[kb] = Quad2{{0u, 0u}};
        if (kb <= QB) {
            f32x4 p;
#pragma unroll
            for (int i = 0; i < 4; i++) p[i] = __builtin_amdgcn_exp2f(st[kb][i] - mx);
            pq[kb] = Act<false>::pack(p);
        }
    }
    f32x4 ot = zero, den = zero;
#pragma unroll
    for (int pp = 0; pp < 2; pp++)
        if (2 * pp <= QB) {
            const bf16x8 bp = join(pq[2 * pp], pq[2 * pp + 1]);
            ot = mfma16(vf[pp], bp, ot);
            den = mfma16(ones, bp, den);
        }
    return ot * __builtin_amdgcn_rcpf(den[0]);
}

// One wave's CPW configurations of a tile (its entries [tb, tb + cnt_w) of
// the class list, cnt_w <= CPW, possibly none: the wave then only takes part
// in the weight hand-over).  NB row blocks from B0 on; Mn: the model of the
// block's next tile, whose first weights are loaded under the last FFN.
template <bool kF8, bool kList, int NB, int B0>
__device__ __forceinline__ void tf_tile(const Bf16View &M, const TfArgs &A, TfLds<kF8> &S, int64_t tb, int cnt_w,
                                        int64_t lbase, const typename Op<kF8>::T *next_w, const float *next_v,
                                        int &vbuf) {
    typedef Op<kF8> OP;
    typedef typename OP::T AT;
    typedef typename OP::Frag Frag;
    constexpr int CPW = NB == 3 ? 1 : 4 / NB, NS = CPW * NB;
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c16 = l & 15, r0 = 4 * (l >> 4), kq = 8 * (l >> 4);
    const uint32_t half0 = l < 32 ? ~0u : 0u, half1 = ~half0;
    const int K = M.K;
    const float *wf = M.wf;
    const int64_t kv_cfg = (int64_t)M.L * (kH / 2) * kKvPerPair;  // cache elements per configuration
    // token of position q (orbital K-1-q) = up bit + 2 down bit, as two
    // wave-uniform 64-bit masks over positions
    uint64_t upm[CPW], dnm[CPW];
    int64_t ent[CPW], smp[CPW];  // list entry (list mode) and sample
#pragma unroll
    for (int c = 0; c < CPW; c++) {
        Key x{0ull, 0ull};
        ent[c] = smp[c] = 0;
        if (c < cnt_w) {
            if (kList) {
                ent[c] = A.list[lbase + tb + c];
                x.lo = A.xkeys[2 * ent[c]];
                x.hi = A.xkeys[2 * ent[c] + 1];
                smp[c] = ent[c] / A.C;
            } else {
                x.lo = A.keys[2 * (tb + c)];
                x.hi = A.keys[2 * (tb + c) + 1];
            }
        }
        const bool inq = l < K;
        upm[c] = __ballot(inq && key_bit(x, 2 * (K - 1 - l)));
        dnm[c] = __ballot(inq && key_bit(x, 2 * (K - 1 - l) + 1));
    }
    auto token = [&](int c, int q) -> int {
        return (int)((upm[c] >> q) & 1ull) | ((int)((dnm[c] >> q) & 1ull) << 1);
    };
    // embeddings of the own rows: tok_emb[prev token] + pos_emb, padding rows 0
    f32x4 h[NS][4];
#pragma unroll
    for (int j = 0; j < NS; j++) {
        const int s = (B0 + j % NB) * 16 + c16;
        const int prev = s == 0 ? 4 : (s < K ? token(j / NB, s - 1) : 0);
#pragma unroll
        for (int db = 0; db < 4; db++) {
            const int c = db * 16 + r0;
            h[j][db] = s < K ? ld4(wf + M.fl.tok_emb + prev * kD + c) + ld4(wf + M.fl.pos_emb + s * kD + c)
                             : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    for (int layer = 0; layer < M.L; layer++) {
        const AT *lw = (kF8 ? reinterpret_cast<const AT *>(M.w8) : reinterpret_cast<const AT *>(M.wb)) +
                       M.bl.layer0 + layer * M.bl.layer_stride;
        weights_ready();  // the attention half and the vectors are here; the last FFN is done
        load_half(S.wf, lw + kAttnElems, kFfnElems, w);
        const float *lv = S.vec[vbuf];
        const float *f8 = lv + kV_f8;  // FP8: power-of-two scale s of each weight matrix and 1/s
        if (cnt_w > 0) {
            Frag x[NS][2];
#pragma unroll
            for (int j = 0; j < NS; j++) normalize<kF8>(h[j], x[j]);
            // the output product's bias; FP8: its products come out scaled by
            // the matrix's power of two s, so the residual is scaled by s
            // around them (exact)
#pragma unroll
            for (int db = 0; db < 4; db++) {
                const f32x4 bo = ld4(lv + kV_bo + db * 16 + r0);
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    h[j][db] += bo;
                    if constexpr (kF8) h[j][db] *= f8[6];
                }
            }
#pragma unroll 1
            for (int hp = 0; hp < 2; hp++) {  // heads 2 hp, 2 hp + 1: one k run of the output product
                typename Act<kF8>::Q op[NS][2];
                // biases of the pair's columns 32 hp + 8 (l >> 4) + 4 t + i (Q, K) and of V's dim c16 of each head
                f32x4 bq[2], bk[2];
                float bv[2];
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    bq[t] = ld4(lv + kV_bqkv + 32 * hp + kq + 4 * t);
                    bk[t] = ld4(lv + kV_bqkv + 64 + 32 * hp + kq + 4 * t);
                    bv[t] = lv[kV_bqkv + 128 + (2 * hp + t) * kDh + c16];
                    if constexpr (kF8) {
                        bq[t] *= f8[0];
                        bk[t] *= f8[2];
                        bv[t] *= f8[4];
                    }
                }
#pragma unroll
                for (int c = 0; c < CPW; c++) {
                    // K operands of both heads (the first head's dims in lanes < 32, the
                    // second's in the others) and V^T operands of each
                    bf16x8 kf[4], vf[2][2];
                    Quad2 vq[2][4];
                    const Quad2 none = {{0u, 0u}};
                    // cached keys [64][32] and values V^T [32][64] of blocks < B0
                    if constexpr (kList && B0 > 0) {
                        const __bf16 *kc = A.kv_in + smp[c] * kv_cfg + ((int64_t)layer * (kH / 2) + hp) * kKvPerPair;
                        const __bf16 *vc = kc + 64 * 2 * kDh;
#pragma unroll
                        for (int kb = 0; kb < B0; kb++)
                            kf[kb] = *reinterpret_cast<const bf16x8 *>(kc + (kb * 16 + c16) * (2 * kDh) + kq);
#pragma unroll
                        for (int hs = 0; hs < 2; hs++) {
                            const __bf16 *vr = vc + (hs * kDh + c16) * 64;
                            if (B0 >= 2) vf[hs][0] = *reinterpret_cast<const bf16x8 *>(vr + kq);
                            if (B0 & 1) vq[hs][B0 - 1] = *reinterpret_cast<const Quad2 *>(vr + (B0 - 1) * 16 + r0);
                        }
                    }
                    {
                        Frag wk[2][2], wv[2][2];
#pragma unroll
                        for (int t = 0; t < 2; t++)
#pragma unroll
                            for (int ks = 0; ks < 2; ks++) {
                                wk[t][ks] = wfrag<kF8>(S.wa, 2 * (4 + 2 * hp + t) + ks);
                                wv[t][ks] = wfrag<kF8>(S.wa, 2 * (8 + 2 * hp + t) + ks);
                            }
#pragma unroll
                        for (int j = 0; j < NB; j++) {
                            const int b = B0 + j;
                            Quad2 k4[2];
#pragma unroll
                            for (int t = 0; t < 2; t++) {
                                f32x4 kt = bk[t], v = f32x4{bv[t], bv[t], bv[t], bv[t]};
#pragma unroll
                                for (int ks = 0; ks < 2; ks++) {
                                    kt = OP::mma(wk[t][ks], x[c * NB + j][ks], kt);
                                    v = OP::mma(x[c * NB + j][ks], wv[t][ks], v);
                                }
                                if constexpr (kF8) {
                                    kt *= f8[3];
                                    v *= f8[5];
                                }
                                k4[t] = Act<false>::pack(kt);
                                vq[t][b] = Act<false>::pack(v);
                            }
                            kf[b] = both(k4[0], k4[1]);
                            if (!kList && A.kv_out && c < cnt_w) {  // keep them for list mode
                                __bf16 *kc = A.kv_out + (tb + c) * kv_cfg + ((int64_t)layer * (kH / 2) + hp) * kKvPerPair;
                                *reinterpret_cast<bf16x8 *>(kc + (b * 16 + c16) * (2 * kDh) + kq) = kf[b];
#pragma unroll
                                for (int t = 0; t < 2; t++)
                                    *reinterpret_cast<Quad2 *>(kc + 64 * 2 * kDh + (t * kDh + c16) * 64 + b * 16 + r0) = vq[t][b];
                            }
                        }
                    }
#pragma unroll
                    for (int hs = 0; hs < 2; hs++)
#pragma unroll
                        for (int pp = 0; 2 * pp < B0 + NB; pp++)
                            if (2 * pp + 1 >= B0)
                                vf[hs][pp] = join(vq[hs][2 * pp], 2 * pp + 1 < B0 + NB ? vq[hs][2 * pp + 1] : none);
                    Frag wq[2][2];
#pragma unroll
                    for (int t = 0; t < 2; t++)
#pragma unroll
                        for (int ks = 0; ks < 2; ks++) wq[t][ks] = wfrag<kF8>(S.wa, 2 * (2 * hp + t) + ks);
#pragma unroll
                    for (int j = 0; j < NB; j++) {
                        Quad2 q4[2];
#pragma unroll
                        for (int t = 0; t < 2; t++) {
                            f32x4 qt = bq[t];
#pragma unroll
                            for (int ks = 0; ks < 2; ks++) qt = OP::mma(wq[t][ks], x[c * NB + j][ks], qt);
                            if constexpr (kF8) qt *= f8[1];
                            q4[t] = Act<false>::pack(qt);
                        }
#pragma unroll
                        for (int hs = 0; hs < 2; hs++)
                            op[c * NB + j][hs] = Act<kF8>::pack(
                                attend(B0 + j, half(both(q4[0], q4[1]), hs ? half1 : half0), kf, vf[hs]));
                    }
                }
                Frag wo[4];
#pragma unroll
                for (int db = 0; db < 4; db++) wo[db] = wfrag<kF8>(S.wa, 24 + 2 * db + hp);
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    const Frag of = join(op[j][0], op[j][1]);
#pragma unroll
                    for (int db = 0; db < 4; db++) h[j][db] = OP::mma(wo[db], of, h[j][db]);
                }
            }
        }
        weights_ready();  // the FFN half is here; the attention half is consumed
        const bool last = layer + 1 == M.L;
        const AT *nw = last ? next_w : lw + M.bl.layer_stride;
        const float *nv = last ? next_v : wf + M.fl.layer0 + (layer + 1) * M.fl.layer_stride;
        if (nw) {
            load_half(S.wa, nw, kAttnElems, w);
            load_half(S.vec[vbuf ^ 1], nv, kVecFloats, w);
        }
        vbuf ^= 1;
        if (cnt_w > 0) {
            Frag x[NS][2];
#pragma unroll
            for (int j = 0; j < NS; j++) {
                if constexpr (kF8) {
#pragma unroll
                    for (int db = 0; db < 4; db++) h[j][db] *= f8[7];
                }
                normalize<kF8>(h[j], x[j]);
                if constexpr (kF8) {
#pragma unroll
                    for (int db = 0; db < 4; db++) h[j][db] *= f8[10];
                }
            }
            // FFN in eight runs of 32 hidden units
#pragma unroll 1
            for (int run = 0; run < 8; run++) {
                Frag w1[2][2];
                f32x4 b1[2];
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    b1[t] = ld4(lv + kV_b1 + run * 32 + kq + 4 * t);
                    if constexpr (kF8) b1[t] *= f8[8];
#pragma unroll
                    for (int ks = 0; ks < 2; ks++) w1[t][ks] = wfrag<kF8>(S.wf, (2 * run + t) * 2 + ks);
                }
                Frag g[NS];
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    typename Act<kF8>::Q gq[2];
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        f32x4 f = b1[t];
#pragma unroll
                        for (int ks = 0; ks < 2; ks++) f = OP::mma(w1[t][ks], x[j][ks], f);
                        f32x4 y;
#pragma unroll
                        for (int i = 0; i < 4; i++) y[i] = gelu_tab(S.gtab, kF8 ? f[i] * f8[9] : f[i]);
                        gq[t] = Act<kF8>::pack(y);
                    }
                    g[j] = both(gq[0], gq[1]);
                }
                Frag w2[4];
#pragma unroll
                for (int db = 0; db < 4; db++) w2[db] = wfrag<kF8>(S.wf, 32 + db * 8 + run);
#pragma unroll
                for (int j = 0; j < NS; j++)
#pragma unroll
                    for (int db = 0; db < 4; db++) h[j][db] = OP::mma(w2[db], g[j], h[j][db]);
            }
#pragma unroll
            for (int db = 0; db < 4; db++) {
                const f32x4 b2 = ld4(lv + kV_b2 + db * 16 + r0);
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    if constexpr (kF8) h[j][db] *= f8[11];
                    h[j][db] += b2;
                }
            }
        }
    }
    if (cnt_w <= 0) return;
    // final LayerNorm (scale folded into the head), head, mask and the
    // log-probability of the actual token, per row block: every lane's group
    // of four lanes holds row c16; lanes 0..15 finish it
    float z[NS][4], rstd[NS], sh[NS];
#pragma unroll
    for (int j = 0; j < NS; j++) {
        row_stats(h[j], rstd[j], sh[j]);
#pragma unroll
        for (int t = 0; t < 4; t++) z[j][t] = 0.f;
    }
#pragma unroll
    for (int db = 0; db < 4; db++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const f32x4 hw4 = ld4(wf + M.fl.head_w + (db * 16 + r0 + i) * 4);
#pragma unroll
            for (int j = 0; j < NS; j++) {
                const float y = fmaf(h[j][db][i], rstd[j], sh[j]);
#pragma unroll
                for (int t = 0; t < 4; t++) z[j][t] = fmaf(y, hw4[t], z[j][t]);
            }
        }
    float slot_lp[NS];
#pragma unroll
    for (int j = 0; j < NS; j++) {
        const int c = j / NB;
#pragma unroll
        for (int t = 0; t < 4; t++) z[j][t] = sum_groups(z[j][t]);
        float lsum = 0.f;
        const int s = (B0 + j % NB) * 16 + c16;
        if (l < 16 && s < K) {
            const uint64_t below = (1ull << s) - 1ull;  // s < K <= 64
            const int up = __popcll(upm[c] & below), dn = __popcll(dnm[c] & below);
            const int rem = K - 1 - s, orb = K - 1 - s;
            float mx = -INFINITY;
            bool ok[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                z[j][t] += wf[M.fl.head_b + t] + wf[M.fl.bias + orb * 4 + t];
                const int bu = t & 1, bd = t >> 1;
                ok[t] = (up + bu <= M.n_up) && (dn + bd <= M.n_dn) && (M.n_up - up - bu <= rem) &&
                        (M.n_dn - dn - bd <= rem);
                if (ok[t]) mx = fmaxf(mx, z[j][t]);
            }
            float den = 0.f;
#pragma unroll
            for (int t = 0; t < 4; t++)
                if (ok[t]) den += __expf(z[j][t] - mx);
            const int ts = token(c, s);
            const float lden = __logf(den);
            const float zt = ts == 0 ? z[j][0] : ts == 1 ? z[j][1] : ts == 2 ? z[j][2] : z[j][3];
            const bool okt = ts == 0 ? ok[0] : ts == 1 ? ok[1] : ts == 2 ? ok[2] : ok[3];
            lsum = okt ? (zt - mx) - lden : -INFINITY;
            if (!kList && A.cond_out && s == A.cond_pos && c < cnt_w)
#pragma unroll
                for (int t = 0; t < 4; t++)
                    A.cond_out[(tb + c) * 4 + t] = ok[t] ? (double)((z[j][t] - mx) - lden) : -INFINITY;
        }
        // the block's rows live in lanes 0..15
        lsum = dpp_row_sum(lsum);
        slot_lp[j] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, lsum)));
    }
    // per configuration: sum of its row blocks in block order
#pragma unroll
    for (int c = 0; c < CPW; c++) {
        if (c >= cnt_w || l != 0) continue;
        if (kList) {
            double acc = A.pre_in[smp[c] * 4 + B0];
#pragma unroll
            for (int b = 0; b < NB; b++) acc += (double)slot_lp[c * NB + b];
            A.xla[ent[c]] = 0.5 * acc;
        } else {
            double acc = 0.0;
#pragma unroll
            for (int b = 0; b < 4; b++) {
                if (A.pre_out) A.pre_out[(tb + c) * 4 + b] = acc;
                if (b < NB) acc += (double)slot_lp[c * NB + b];
            }
            A.logabs[tb + c] = 0.5 * acc;
        }
    }
}

// Configurations per wave of a class whose x' have nb row blocks of their own.
__device__ __forceinline__ int cfgs_per_wave(int nb) { return nb <= 1 ? 4 : nb == 2 ? 2 : 1; }

// Persistent loop over tiles.  A tile holds the configurations of `wpt`
// waves, all of one class (and one item of a batched launch): eight where
// that still gives every CU a tile, fewer for small work, so that it spreads
// over more CUs (a wave's time hardly depends on its neighbours').
template <bool kList, bool kF8, bool kBatch>
__device__ __forceinline__ void transformer(const Bf16View &M0, const TfArgs &A0, const TfItem *items, int n_items) {
    typedef Op<kF8> OP;
    typedef typename OP::T AT;
    __shared__ __align__(16) TfLds<kF8> S;
    // first tile of every (item, class), in item-major order
    __shared__ int64_t sh_tile0[kBatch ? 4 * kMaxTfItems + 1 : 5], sh_cnt[kBatch ? 4 * kMaxTfItems : 4];
    __shared__ int sh_blocks[kBatch ? 4 * kMaxTfItems : 4];
    __shared__ int sh_wpt;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nq = kBatch ? 4 * n_items : kList ? 4 : 1;  // (item, class) pairs
    auto count = [&](int q) -> int64_t {
        if (kBatch) return items[q >> 2].A.hdr[q & 3];
        return kList ? A0.hdr[q] : A0.n;
    };
    auto blocks_of = [&](int q) -> int {  // row blocks a configuration of the pair evaluates
        const int K = kBatch ? items[q >> 2].M.K : M0.K;
        // batch sampling reads one position's conditionals: later rows do not reach it
        const int rows = !kList && A0.cond_out ? A0.cond_pos + 1 : K;
        return ((rows + 15) >> 4) - (kList ? (q & 3) : 0);
    };
    for (int i = threadIdx.x; i < kGeluN; i += blockDim.x)  // the same table in every model
        S.gtab[i] = make_float2(M0.wf[M0.fl.gelu + 2 * i], M0.wf[M0.fl.gelu + 2 * i + 1]);
    for (int q = threadIdx.x; q < nq; q += blockDim.x) {
        sh_cnt[q] = count(q);
        sh_blocks[q] = blocks_of(q);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t units = 0;
        for (int q = 0; q < nq; q++) {
            const int cpw = cfgs_per_wave(sh_blocks[q]);
            units += (sh_cnt[q] + cpw - 1) / cpw;
        }
        int64_t wpt = (units + gridDim.x - 1) / gridDim.x;
        wpt = wpt < 1 ? 1 : wpt > kTfWaves ? kTfWaves : wpt;
        int64_t acc = 0;
        for (int q = 0; q < nq; q++) {
            const int64_t per = wpt * cfgs_per_wave(sh_blocks[q]);
            sh_tile0[q] = acc;
            acc += (sh_cnt[q] + per - 1) / per;
        }
        sh_tile0[nq] = acc;
        sh_wpt = (int)wpt;
    }
    __syncthreads();
    const int64_t T = sh_tile0[nq];
    const int wpt = sh_wpt;
    auto pair_of = [&](int64_t tile) -> int {  // the last pair whose first tile is at or before `tile`
        int q = 0;
        if (kBatch) {
            for (int step = 4 * kMaxTfItems; step >= 1; step >>= 1)
                if (q + step < nq && sh_tile0[q + step] <= tile) q += step;
        } else if (kList) {
            for (int c = 1; c < 4; c++)
                if (sh_tile0[c] <= tile) q = c;
        }
        return __builtin_amdgcn_readfirstlane(q);
    };
    auto weights_of = [&](const Bf16View &M) -> const AT * {
        return (kF8 ? reinterpret_cast<const AT *>(M.w8) : reinterpret_cast<const AT *>(M.wb)) + M.bl.layer0;
    };
    if ((int64_t)blockIdx.x >= T) return;
    int q = pair_of(blockIdx.x);
    int vbuf = 0;
    {
        const Bf16View &M = kBatch ? items[q >> 2].M : M0;
        load_half(S.wa, weights_of(M), kAttnElems, w);
        load_half(S.vec[0], M.wf + M.fl.layer0, kVecFloats, w);
    }
    for (int64_t tile = blockIdx.x; tile < T; tile += gridDim.x) {
        const int64_t next = tile + gridDim.x;
        const int qn = next < T ? pair_of(next) : q;
        const Bf16View &Mn = kBatch ? items[qn >> 2].M : M0;
        const AT *next_w = next < T ? weights_of(Mn) : nullptr;
        const float *next_v = Mn.wf + Mn.fl.layer0;
        const Bf16View M = kBatch ? items[q >> 2].M : M0;
        const TfArgs A = kBatch ? items[q >> 2].A : A0;
        const int cls = kList ? (q & 3) : 0;
        const int nb = __builtin_amdgcn_readfirstlane(sh_blocks[q]), cpw = cfgs_per_wave(nb);
        const int64_t cnt = sh_cnt[q], tb = ((tile - sh_tile0[q]) * wpt + w) * cpw;
        const int64_t left = w < wpt ? cnt - tb : 0;
        const int cnt_w = __builtin_amdgcn_readfirstlane((int)(left < 0 ? 0 : left < cpw ? left : cpw));
        const int64_t lbase = kList ? A.hdr[4 + cls] : 0;
#define NNQS_TILE(NB, B0) tf_tile<kF8, kList, NB, B0>(M, A, S, tb, cnt_w, lbase, next_w, next_v, vbuf)
        if constexpr (kList) {
            switch (nb * 4 + cls) {
                case 16: NNQS_TILE(4, 0); break;
                case 12: NNQS_TILE(3, 0); break;
                case 13: NNQS_TILE(3, 1); break;
                case 8: NNQS_TILE(2, 0); break;
                case 9: NNQS_TILE(2, 1); break;
                case 10: NNQS_TILE(2, 2); break;
                case 4: NNQS_TILE(1, 0); break;
                case 5: NNQS_TILE(1, 1); break;
                case 6: NNQS_TILE(1, 2); break;
                case 7: NNQS_TILE(1, 3); break;
                default:  // no row of its own (the sample itself, K a multiple of 16): the prefix sum
                    if ((threadIdx.x & 63) < (unsigned)cnt_w) {
                        const int64_t e = A.list[lbase + tb + (threadIdx.x & 63)];
                        A.xla[e] = 0.5 * A.pre_in[(e / A.C) * 4 + cls];
                    }
                    if (kBatch && next_w) {  // the weights in LDS are this item's; the next tile may be another's
                        weights_ready();
                        load_half(S.wa, next_w, kAttnElems, w);
                        load_half(S.vec[vbuf], next_v, kVecFloats, w);
                    }
            }
        } else {
            switch (nb) {
                case 4: NNQS_TILE(4, 0); break;
                case 3: NNQS_TILE(3, 0); break;
                case 2: NNQS_TILE(2, 0); break;
                default: NNQS_TILE(1, 0); break;
            }
        }
#undef NNQS_TILE
        q = qn;
    }
}


// Launches (transformer_*.hip); grid: blocks of kTfWaves waves.
void tf_launch_sample(bool fp8, unsigned grid, hipStream_t st, const Bf16View &M, const TfArgs &A);
void tf_launch_list(bool fp8, unsigned grid, hipStream_t st, const Bf16View &M, const TfArgs &A);
// One position of batch sampling (transformer_rows.hip): conditionals of
// position s for n prefixes.
struct RowPtrs {
    __bf16 *p[64];  // per position: the rows of its prefixes ([L][2 pairs of heads][K 32 | V 32] each)
};
struct RowsArgs {
    const uint64_t *keys;   // [n][2], bits of the tokens before s
    const int32_t *path;    // [n][64]: the prefix's ancestor among those of position i < s
    int64_t n;
    int s, per;             // per: prefixes per wave (set by the launch)
    double *cond;           // [n][4]
    RowPtrs rows;           // rows of positions < s read, of s written
};
nnqs_status tf_launch_rows(int cus, hipStream_t st, const Bf16View &M, RowsArgs A);
size_t rows_entry_bytes(int n_layers);  // of one prefix's row
nnqs_status enqueue_bf16_rows(const nnqs_model *m, const RowsArgs &A, hipStream_t st);
nnqs_status enqueue_phase_bf16(const nnqs_model *m, const uint64_t *keys, int64_t n, double *phase, hipStream_t st);
void tf_launch_batch(unsigned grid, hipStream_t st, const Bf16View &M0, const TfItem *items, int n_items);

}  // namespace nnqs
