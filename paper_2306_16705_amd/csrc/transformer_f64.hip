// FP64 forward of the amplitude transformer (Section 3.1, Eq. 11, Fig. 2;
// d_model 64, 4 heads, any FFN width that is a multiple of 64) in one launch.
//
// A wave owns one block of 16 sequence rows of one configuration and keeps
// it in registers through all layers, transposed: lane l = 16 lk + lr holds
// row lr and, of column tile t, columns 16 t + lk + 4 i, i = 0..3.  On
// v_mfma_f64_16x16x4_f64 the accumulator layout (rows lk + 4 i, column lr) is
// the operand layout of the next product (k = 4 k4 + lk with k4 = 4 t + i,
// row or column lr), so tiles pass from product to product as they are:
// normalised rows -> Q, K, V -> scores -> probabilities -> attention output ->
// residual -> hidden units -> residual.  Four waves form a block, the row
// blocks of 4 / nb configurations of nb row blocks each, and two blocks share
// a CU; K and V of a head go through LDS to the configuration's other waves.
//
// Weights stream through LDS in steps of 16 KB, 32 fragments of 16 x 4 in
// operand order (512 B each, conflict-free): a head's W_k and W_v, then its
// W_q and rows of W_o, then 16 hidden units of W1 and W2 at a time.  They come
// from a copy of the master weights packed in that order (k64_pack) by
// global_load_lds, the next step's in flight under the current one, with one
// barrier per step.
//
// Bound: FP64 MFMA (K = 60: 27.8 MFLOP per configuration, 64 of whose rows
// are run for 60).  Against one kernel per product with the rows in memory
// between them (about 11 KB of traffic per row and layer), one MI355X, whole
// calls: log|psi| and phase of 1,001 configurations at K = 60 1,118 -> 671 us;
// FP64 E_loc of 8 samples at K = 16 (25,544 x') 9,544 -> 4,215 us (680 and 4,276
// us with the products summed into the residual, twice the rounding error of
// log|psi|).  Matrix
// products alone (no softmax, GELU, LayerNorm or loads) take 70 % of the
// present time: FP64 vector work adds to them (GELU 9 %, attention 16 % of
// it), as does the latency of each step's barrier; eight or twelve waves in
// lockstep per block were 8 and 19 % slower, three blocks per CU (168
// registers) 2 % slower.  At the 256 registers of two blocks some addresses
// spill (224 bytes a lane, 264 in list mode).
#include <cmath>

#include "f64_kernels.hpp"

namespace nnqs {

constexpr int kW64 = 4;                   // waves per block (one per SIMD, two blocks per CU)
constexpr int kFrag = 64;                 // doubles of one operand fragment
constexpr int kStepDoubles = 32 * kFrag + 128;  // one step's fragments and bias vectors (17 KB)
constexpr int kKvTile = 256;              // one head's K or V of 16 rows, in operand order

struct T64Args {
    const uint64_t *keys;  // sample mode: configurations
    int64_t n;
    double *logabs;
    const double *packed;  // the layers' weights as k64_pack leaves them
    double *kv_out;   // sample mode: cache written (may be null): [L][4 heads][K, V][row blocks][256] per configuration
    double *pre_out;  // prefix sums of log pi over the first 16 b positions, b = 0..3 (with kv_out)
    const double *kv_in;   // list mode
    const double *pre_in;
    const int32_t *list;
    const int64_t *hdr;  // {count[4], offset[4]} by first row block
    const uint64_t *xkeys;
    int64_t C;
    double *xla;
    int cond_pos;      // sample mode: position whose conditionals are written
    double *cond_out;  // [n][4] (may be null)
};

constexpr int kParked = 14;  // of a lane's 16 residual values; all 16 would leave room for one block per CU

struct T64Lds {
    double w[2][kStepDoubles];
    double kv[kW64][2][kKvTile];
    double park[kW64][kParked][64];  // each lane's own: no wait but its own
    double lp[kW64];
    int64_t tile0[5], cnt[4];
    int cpt[4];
};

// A double with that of the lane group 16 (32) lanes away, in either order.
struct DPair {
    double a, b;
};
template <bool k32>
__device__ __forceinline__ DPair swap_groups(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    uint32_t a0, a1, b0, b1;
    if constexpr (k32) {
        const auto p = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto q = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        a0 = p[0], b0 = p[1], a1 = q[0], b1 = q[1];
    } else {
        const auto p = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto q = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        a0 = p[0], b0 = p[1], a1 = q[0], b1 = q[1];
    }
    return {__builtin_bit_cast(double, ((uint64_t)a1 << 32) | a0), __builtin_bit_cast(double, ((uint64_t)b1 << 32) | b0)};
}
__device__ __forceinline__ double xor_sum(double v) {  // over lk: lanes l, l ^ 16, l ^ 32, l ^ 48
    const DPair p = swap_groups<false>(v);
    const DPair q = swap_groups<true>(p.a + p.b);
    return q.a + q.b;
}
__device__ __forceinline__ double xor_max(double v) {
    const DPair p = swap_groups<false>(v);
    const DPair q = swap_groups<true>(fmax(p.a, p.b));
    return fmax(q.a, q.b);
}

__device__ __forceinline__ f64x4 mma64(double a, double b, const f64x4 &c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// LayerNorm of the wave's rows (two-pass statistics, eps 1e-5).
__device__ __forceinline__ void layernorm64(const f64x4 (&h)[4], const double *__restrict__ g,
                                            const double *__restrict__ b, uint32_t lk, f64x4 (&x)[4]) {
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
        for (int i = 0; i < 4; i++) s += h[t][i];
    const double mean = xor_sum(s) / 64.0;
    double q = 0.0;
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
        for (int i = 0; i < 4; i++) q += (h[t][i] - mean) * (h[t][i] - mean);
    const double r = 1.0 / sqrt(xor_sum(q) / 64.0 + 1e-5);
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t c = 16 * t + 4 * i + lk;
            x[t][i] = (h[t][i] - mean) * r * g[c] + b[c];
        }
}

// Steps of a layer: 2 hh and 2 hh + 1 for head hh, then F / 16 of the FFN.
// Fragments (k4 = 0 .. 15, t = 0 .. 3; element [lk][lr] is row 4 k4 + lk,
// column lr of a 64 x 16 slice, or of rows and column block t) and vectors (the
// last of each sum with the sum's bias from kSumBias on):
//  2 hh:     k4: W_k, 16 + k4: W_v of the head's columns; b_k, b_v
//  2 hh + 1: k4: W_q of the head's columns; 16 + 4 i + t: W_o rows 16 hh + 4 i ..; b_q, b_o
//  8 + u:    k4: W1 of hidden units 16 u ..; 16 + 4 i + t: W2 rows 16 u + 4 i ..; b1, b2
constexpr int kSumBias = 32 * kFrag + 64;
__host__ __device__ inline int f64_steps(int F) { return 8 + F / 16; }

__global__ void __launch_bounds__(256) k64_pack(ModelView M, double *__restrict__ out) {
    const int steps = f64_steps(M.F);
    const LayerOffsets o = layer_offsets(64, M.F);
    const int layer = blockIdx.x / steps, s = blockIdx.x % steps;
    const double *W = M.w64 + M.off.layer0 + (int64_t)layer * M.off.layer_stride;
    double *dst = out + (int64_t)blockIdx.x * kStepDoubles;
    for (int e = threadIdx.x; e < kStepDoubles; e += 256) {
        const int f = e >> 6, lk = (e >> 4) & 3, lr = e & 15;
        int64_t src = -1;
        if (e >= 32 * kFrag) {
            const int v = e - 32 * kFrag;
            if (e >= kSumBias) src = s == 7 ? o.bo + e - kSumBias : s == steps - 1 ? o.b2 + e - kSumBias : -1;
            else if (s >= 8) src = v < 16 ? o.b1 + 16 * (s - 8) + v : -1;
            else if (s & 1) src = v < 16 ? o.bq + 8 * (s - 1) + v : -1;
            else src = v < 16 ? o.bk + 8 * s + v : v < 32 ? o.bv + 8 * s + v - 16 : -1;
        } else {
            const int k = 4 * (f & 15) + lk;                        // row of a 64 x 16 slice
            const int i = (f - 16) >> 2, c = 16 * (f & 3) + lr;     // 16 rows x 64 columns
            if (s >= 8) src = f < 16 ? o.w1 + (int64_t)k * M.F + 16 * (s - 8) + lr : o.w2 + (int64_t)(16 * (s - 8) + 4 * i + lk) * 64 + c;
            else if (s & 1) src = f < 16 ? o.wq + k * 64 + 8 * (s - 1) + lr : o.wo + (8 * (s - 1) + 4 * i + lk) * 64 + c;
            else src = (f < 16 ? o.wk : o.wv) + k * 64 + 8 * s + lr;
        }
        dst[e] = src >= 0 ? W[src] : 0.0;
    }
}

// Loads one packed step: 17 pieces of 1 KB dealt to the waves in turn.
__device__ __forceinline__ void load_step(double *dst, const double *__restrict__ src, int w) {
    const uint32_t l = threadIdx.x & 63;
    for (int p = w; p < 17; p += kW64)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + 128 * p + 2 * l),
                                         (__attribute__((address_space(3))) void *)(dst + 128 * p), 16, 0, 0);
}

// Causal attention of query block QB for one head (kv: K or V tile of a key
// block): o = V^T exp(scale (S - max)) (taken as 2^x), den = this lane's share of the sums.
template <int QB, typename KV>
__device__ __forceinline__ void attend64(const KV &kv, const f64x4 &qt, uint32_t lk, uint32_t lr, f64x4 &o, double &den) {
    f64x4 st[QB + 1];
    // scores S^T[key][query]: register i of block kb is key 16 kb + 4 i + lk
    f64x4 kf = kv(0, 0);
#pragma unroll
    for (int kb = 0; kb <= QB; kb++) {
        const f64x4 kn = kb < QB ? kv(kb + 1, 0) : kf;
        st[kb] = f64x4{0.0, 0.0, 0.0, 0.0};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; i++) st[kb] = mma64(kf[i], qt[i], st[kb]);
        kf = kn;
    }
    double mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb <= QB; kb++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if (kb == QB && 4 * i + lk > lr) st[kb][i] = -INFINITY;  // a later key
            mx = fmax(mx, st[kb][i]);
        }
    f64x4 vf = kv(0, 1);
    mx = xor_max(mx);
    constexpr double kScale = 0.25 * 1.4426950408889634;  // 1 / sqrt(64 / 4 heads), in base 2
    const double off = -mx * kScale;
    ConstF64 *tab = exp2_table();
    den = 0.0;
    o = f64x4{0.0, 0.0, 0.0, 0.0};
    f64x4 o2 = o;
#pragma unroll
    for (int kb = 0; kb <= QB; kb++) {
        const f64x4 vn = kb < QB ? kv(kb + 1, 1) : vf;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const double p = exp2_f64(tab, fma(st[kb][i], kScale, off));
            den += p;
            if (i & 1) o2 = mma64(vf[i], p, o2);
            else o = mma64(vf[i], p, o);
        }
        vf = vn;
    }
    o += o2;
}

// a + b += (64 x 16 slice in fragments 0 .. 15)^T x, even and odd k4 apart.
__device__ __forceinline__ void project(const double *wb, const f64x4 (&x)[4], uint32_t l, f64x4 &a, f64x4 &b) {
    double wn[3][4];
    auto read = [&](int g) {
#pragma unroll
        for (int e = 0; e < 4; e++) wn[g % 3][e] = wb[(4 * g + e) * kFrag + l];
    };
    read(0);
    read(1);
#pragma unroll
    for (int g = 0; g < 4; g++) {
        if (g + 2 < 4) read(g + 2);
        __builtin_amdgcn_sched_barrier(0);
        a = mma64(wn[g % 3][0], x[g][0], a);
        b = mma64(wn[g % 3][1], x[g][1], b);
        a = mma64(wn[g % 3][2], x[g][2], a);
        b = mma64(wn[g % 3][3], x[g][3], b);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// h += (16 x 64 rows in fragments 16 .. 31)^T v.
__device__ __forceinline__ void add_rows(const double *wb, const f64x4 &v, uint32_t l, f64x4 (&h)[4]) {
    double wn[2][4];
#pragma unroll
    for (int t = 0; t < 4; t++) wn[0][t] = wb[(16 + t) * kFrag + l];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (i + 1 < 4)
#pragma unroll
            for (int t = 0; t < 4; t++) wn[(i + 1) & 1][t] = wb[(16 + 4 * (i + 1) + t) * kFrag + l];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; t++) h[t] = mma64(wn[i & 1][t], v[i], h[t]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ __forceinline__ void step_ready() {  // this wave's pieces have arrived, then everyone's
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

template <bool kList>
__device__ __forceinline__ void transformer_f64(const ModelView &M, const T64Args &A) {
    __shared__ __align__(16) T64Lds S;
    const uint32_t l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lr = l & 15, lk = l >> 4;
    const int K = M.K, F = M.F, L = M.L;
    const LayerOffsets LO = layer_offsets(64, F);
    const double *W = M.w64;
    const int steps = f64_steps(F);  // per layer
    const int64_t total = (int64_t)L * steps * kStepDoubles;
    // rows that reach the result: all, or up to the position whose conditionals are asked for
    const int rows = !kList && A.cond_out ? A.cond_pos + 1 : K;
    const int nb_all = (rows + 15) >> 4;
    const int64_t kv_head = 2 * nb_all * kKvTile;  // cached K and V of one head and layer (written for whole rows only)
    if (threadIdx.x < 4) S.cnt[threadIdx.x] = kList ? A.hdr[threadIdx.x] : threadIdx.x == 0 ? A.n : 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t acc = 0;
        for (int q = 0; q < 4; q++) {
            const int nb = nb_all - q;
            S.cpt[q] = nb <= 0 ? 64 * kW64 : kW64 / nb;  // configurations per tile
            S.tile0[q] = acc;
            acc += (S.cnt[q] + S.cpt[q] - 1) / S.cpt[q];
        }
        S.tile0[4] = acc;
    }
    __syncthreads();
    const int64_t T = S.tile0[4];
    if ((int64_t)blockIdx.x >= T) return;
    int buf = 0;
    load_step(S.w[0], A.packed, w);
    int64_t at = 0;  // the step in S.w[buf]
    auto next_step = [&](bool more) {  // loads the step after `at` (the first one again after the last)
        at += kStepDoubles;
        if (at == total) at = 0;
        if (more) load_step(S.w[buf ^ 1], A.packed + at, w);
    };
    for (int64_t tile = blockIdx.x; tile < T; tile += gridDim.x) {
        int q = 0;
        for (int c = 1; c < 4; c++)
            if (S.tile0[c] <= tile) q = c;
        q = __builtin_amdgcn_readfirstlane(q);
        const int b0 = kList ? q : 0, nb = nb_all - b0, cpt = __builtin_amdgcn_readfirstlane(S.cpt[q]);
        const int64_t tb = (tile - S.tile0[q]) * cpt;  // first configuration of the tile in its class
        const int64_t left = S.cnt[q] - tb;
        const int ncfg = __builtin_amdgcn_readfirstlane((int)(left < cpt ? left : cpt));
        const int64_t lbase = kList ? A.hdr[4 + q] : 0;
        if (nb <= 0) {  // no row of its own (the sample itself, K a multiple of 16)
            if ((int)threadIdx.x < ncfg) {
                const int64_t e = A.list[lbase + tb + threadIdx.x];
                A.xla[e] = 0.5 * A.pre_in[(e / A.C) * 4 + b0];
            }
            continue;  // the weights in LDS stay the first step's
        }
        // The wave's configuration and row block.  With three row blocks a wave
        // has none; which one turns with the block, so that no SIMD is left out.
        const int role = nb == 3 ? (w + (int)blockIdx.x) & 3 : w;
        const int c = role / nb, QB = b0 + role % nb;
        const bool on = c < ncfg;  // wave-uniform
        Key x{0ull, 0ull};
        int64_t ent = 0, smp = 0;
        if (on) {
            if (kList) {
                ent = A.list[lbase + tb + c];
                x.lo = A.xkeys[2 * ent];
                x.hi = A.xkeys[2 * ent + 1];
                smp = ent / A.C;
            } else {
                x.lo = A.keys[2 * (tb + c)];
                x.hi = A.keys[2 * (tb + c) + 1];
            }
        }
        // token of position p (orbital K-1-p) = up bit + 2 down bit
        const uint64_t upm = __ballot((int)l < K && key_bit(x, 2 * (K - 1 - (int)l)));
        const uint64_t dnm = __ballot((int)l < K && key_bit(x, 2 * (K - 1 - (int)l) + 1));
        auto token = [&](int p) { return (int)((upm >> p) & 1ull) | ((int)((dnm >> p) & 1ull) << 1); };
        const int s = 16 * QB + (int)lr;  // the lane's position
        f64x4 h[4];
        {
            const int prev = s == 0 ? 4 : s < K ? token(s - 1) : 0;
            const double *te = W + M.off.tok_emb, *pe = W + M.off.pos_emb;
            uint32_t lv = lk;
            asm volatile("" : "+v"(lv));
            const uint32_t to = prev * 64 + lv, po = (s < K ? s : 0) * 64 + lv;
#pragma unroll
            for (int t = 0; t < 4; t++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const double e = te[to + 16 * t + 4 * i] + pe[po + 16 * t + 4 * i];
                    h[t][i] = s < K ? e : 0.0;
                }
        }
        for (int layer = 0; layer < L; layer++) {
            const double *Lw = W + M.off.layer0 + (int64_t)layer * M.off.layer_stride;
            uint32_t lv = lk;  // a fresh value per layer: the vectors' addresses are not kept in registers
            asm volatile("" : "+v"(lv));
            f64x4 xn[4];
            // A product that goes into the residual is summed in h from zero while
            // the residual waits, and added to it once with its bias: summed into
            // the residual itself, every step would round at the residual's size.
            double kept[16 - kParked];
            auto park = [&] {
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    if (e < kParked) S.park[w][e][l] = h[e >> 2][e & 3];
                    else kept[e - kParked] = h[e >> 2][e & 3];
                    h[e >> 2][e & 3] = 0.0;
                }
            };
            auto unpark = [&] {
                const double *bias = S.w[buf ^ 1] + kSumBias;  // the step just done, until the next one is ready
#pragma unroll
                for (int e = 0; e < 16; e++)
                    h[e >> 2][e & 3] = (e < kParked ? S.park[w][e][l] : kept[e - kParked]) + (bias[4 * e + lk] + h[e >> 2][e & 3]);
            };
            if (on) {
                layernorm64(h, Lw + LO.ln1_g, Lw + LO.ln1_b, lv, xn);
                park();
            }
#pragma unroll 1
            for (int hh = 0; hh < 4; hh++) {
                step_ready();
                const double *wb = S.w[buf];
                next_step(true);
                buf ^= 1;
                if (on) {
                    f64x4 kt, v;
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        kt[i] = wb[32 * kFrag + 4 * i + lk];
                        v[i] = wb[32 * kFrag + 16 + lr];
                    }
                    // operands are read two groups ahead of their products (the
                    // compiler alone reads each just before it is needed)
                    double wn[3][4];
                    auto read = [&](int g) {
#pragma unroll
                        for (int e = 0; e < 4; e++) wn[g % 3][e] = wb[(16 * (e & 1) + 2 * g + (e >> 1)) * kFrag + l];
                    };
                    read(0);
                    read(1);
#pragma unroll
                    for (int g = 0; g < 8; g++) {
                        if (g + 2 < 8) read(g + 2);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int e = 0; e < 2; e++) {
                            const double xv = xn[g >> 1][2 * (g & 1) + e];
                            kt = mma64(wn[g % 3][2 * e], xv, kt);
                            v = mma64(xv, wn[g % 3][2 * e + 1], v);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    *reinterpret_cast<f64x4 *>(S.kv[role][0] + 4 * l) = kt;
                    *reinterpret_cast<f64x4 *>(S.kv[role][1] + 4 * l) = v;
                    if (!kList && A.kv_out) {
                        double *dst = A.kv_out + (((tb + c) * L + layer) * 4 + hh) * kv_head + QB * kKvTile + 4 * l;
                        *reinterpret_cast<f64x4 *>(dst) = kt;
                        *reinterpret_cast<f64x4 *>(dst + nb_all * kKvTile) = v;
                    }
                }
                step_ready();  // also: K and V of every row block written
                wb = S.w[buf];
                next_step(true);
                buf ^= 1;
                if (on) {
                    f64x4 qt, q2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int i = 0; i < 4; i++) qt[i] = wb[32 * kFrag + 4 * i + lk];
                    project(wb, xn, l, qt, q2);
                    qt += q2;
                    const double *kvc = kList ? A.kv_in + ((smp * L + layer) * 4 + hh) * kv_head : nullptr;
                    auto kv_tile = [&](int kb, int which) -> f64x4 {
                        if (kList && kb < b0) return *reinterpret_cast<const f64x4 *>(kvc + (nb_all * which + kb) * kKvTile + 4 * l);
                        return *reinterpret_cast<const f64x4 *>(S.kv[c * nb + kb - b0][which] + 4 * l);
                    };
                    f64x4 o;
                    double den;
                    switch (QB) {  // wave-uniform; straight-line code for each count of key blocks
                        case 0: attend64<0>(kv_tile, qt, lk, lr, o, den); break;
                        case 1: attend64<1>(kv_tile, qt, lk, lr, o, den); break;
                        case 2: attend64<2>(kv_tile, qt, lk, lr, o, den); break;
                        default: attend64<3>(kv_tile, qt, lk, lr, o, den); break;
                    }
                    o *= 1.0 / xor_sum(den);
                    add_rows(wb, o, l, h);
                }
            }
            if (on) {
                unpark();
                layernorm64(h, Lw + LO.ln2_g, Lw + LO.ln2_b, lv, xn);
                park();
            }
#pragma unroll 1
            for (int sp = 8; sp < steps; sp++) {
                step_ready();
                const double *wb = S.w[buf];
                next_step(sp + 1 < steps || layer + 1 < L || tile + gridDim.x < T);
                buf ^= 1;
                if (on) {
                    f64x4 f, f2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int i = 0; i < 4; i++) f[i] = wb[32 * kFrag + 4 * i + lk];
                    project(wb, xn, l, f, f2);
                    double g[4];
#pragma unroll
                    for (int i = 0; i < 4; i++) g[i] = f[i] + f2[i];
                    gelu_f64_set(g);
                    add_rows(wb, f64x4{g[0], g[1], g[2], g[3]}, l, h);
                }
            }
            if (on) unpark();
        }
        // final LayerNorm, head, mask (Eq. 12, read with the lower bound too)
        // and the log-probability of the actual token
        if (on) {
            f64x4 xn[4];
            uint32_t lv = lk;
            asm volatile("" : "+v"(lv));
            layernorm64(h, W + M.off.lnf_g, W + M.off.lnf_b, lv, xn);
            double z[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int t = 0; t < 4; t++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const f64x4 hw = *reinterpret_cast<const f64x4 *>(W + M.off.head_w + (16 * t + 4 * i + lv) * 4);
#pragma unroll
                    for (int u = 0; u < 4; u++) z[u] += xn[t][i] * hw[u];
                }
#pragma unroll
            for (int u = 0; u < 4; u++) z[u] = xor_sum(z[u]);
            double lp = 0.0;
            if (l < 16 && s < K) {
                const uint64_t below = (1ull << s) - 1ull;  // s < K <= 64
                const int up = __popcll(upm & below), dn = __popcll(dnm & below);
                const int rem = K - 1 - s;
                bool ok[4];
                double mx = -INFINITY;
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    z[u] += W[M.off.head_b + u] + W[M.off.bias + rem * 4 + u];  // position s holds orbital K-1-s
                    const int bu = u & 1, bd = u >> 1;
                    ok[u] = (up + bu <= M.n_up) && (dn + bd <= M.n_dn) && (M.n_up - up - bu <= rem) &&
                            (M.n_dn - dn - bd <= rem);
                    if (ok[u] && z[u] > mx) mx = z[u];
                }
                double den = 0.0;
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (ok[u]) den += exp(z[u] - mx);
                const double lden = log(den);
                const int ts = token(s);
                lp = -INFINITY;
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (u == ts && ok[u]) lp = (z[u] - mx) - lden;
                if (!kList && A.cond_out && s == A.cond_pos)
#pragma unroll
                    for (int u = 0; u < 4; u++) A.cond_out[(tb + c) * 4 + u] = ok[u] ? (z[u] - mx) - lden : -INFINITY;
            }
            // the rows' sum over lanes 0..15 (lanes of a group differ in lr only)
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) lp += __shfl_xor(lp, off, 64);
            if (l == 0) S.lp[role] = lp;
        }
        __syncthreads();
        if ((int)threadIdx.x < ncfg) {  // row blocks in order
            const int cc = threadIdx.x;
            if (kList) {
                const int64_t e = A.list[lbase + tb + cc];
                double acc = A.pre_in[(e / A.C) * 4 + b0];
                for (int b = 0; b < nb; b++) acc += S.lp[cc * nb + b];
                A.xla[e] = 0.5 * acc;
            } else {
                double acc = 0.0;
                for (int b = 0; b < 4; b++) {
                    if (A.pre_out) A.pre_out[(tb + cc) * 4 + b] = acc;
                    if (b < nb) acc += S.lp[cc * nb + b];
                }
                A.logabs[tb + cc] = 0.5 * acc;
            }
        }
    }
}

__global__ void __launch_bounds__(64 * kW64, 2) k64_transformer(ModelView M, T64Args A) { transformer_f64<false>(M, A); }

__global__ void __launch_bounds__(64 * kW64, 2) k64_transformer_list(ModelView M, T64Args A) { transformer_f64<true>(M, A); }

int64_t f64_cache_doubles(const nnqs_model *m) {
    return (int64_t)m->desc.n_layers * 4 * 2 * ((m->desc.n_orb + 15) / 16) * kKvTile;
}

static unsigned grid64(int64_t n) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    return (unsigned)(n < 1 ? 1 : n < 2 * cus ? n : 2 * cus);  // two blocks per CU (256 registers, 52 KB of LDS)
}

size_t f64_packed_bytes(const nnqs_model_desc &d) {
    return (size_t)d.n_layers * f64_steps(d.d_ff) * kStepDoubles * sizeof(double);
}

void f64_pack(const ModelView &M, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k64_pack, dim3((unsigned)(M.L * f64_steps(M.F))), dim3(256), 0, st, M, out);
}

void transformer_f64_sample(const ModelView &M, const double *packed, const uint64_t *keys, int64_t n, double *logabs,
                            int cpos, double *cond, double *kvc, double *pre, hipStream_t st) {
    T64Args A{};
    A.packed = packed;
    A.keys = keys;
    A.n = n;
    A.logabs = logabs;
    A.cond_pos = cpos;
    A.cond_out = cond;
    A.kv_out = kvc;
    A.pre_out = pre;
    hipLaunchKernelGGL(k64_transformer, dim3(grid64(n)), dim3(64 * kW64), 0, st, M, A);
}

void transformer_f64_list(const ModelView &M, const double *packed, const uint64_t *xkeys, int64_t C,
                          const int32_t *list, const int64_t *hdr, int64_t n, const double *kvc, const double *pre,
                          double *xla, hipStream_t st) {
    T64Args A{};
    A.packed = packed;
    A.xkeys = xkeys;
    A.C = C;
    A.list = list;
    A.hdr = hdr;
    A.kv_in = kvc;
    A.pre_in = pre;
    A.xla = xla;
    hipLaunchKernelGGL(k64_transformer_list, dim3(grid64(n)), dim3(64 * kW64), 0, st, M, A);
}

}  // namespace nnqs
