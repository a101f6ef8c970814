// One position of batch sampling: the BF16 transformer's row s of every unique
// prefix, with the keys and values of the rows before it read from where their
// own positions left them (rows.p[i], one entry per prefix of position i, found
// through the prefix's path).
#include "transformer.hpp"

namespace nnqs {

// A wave takes up to 16 prefixes, one row each, in the layout of tf_tile with
// prefixes in the place of a block's rows: every product of the layer serves
// 16 prefixes.  Only attention differs: the keys and values are each prefix's
// own, so the score product runs once per prefix on its keys and only that
// prefix's column is taken from it (an infinity or NaN among one prefix's keys
// and values stays its own), and so does the value product.  The softmax runs
// once for all 16.  Values come as
// rows; a product with an identity makes the untransposed tile that tf_tile
// holds.  Products, sums and their order per row are those of the whole
// forward, so the conditionals are the same bits.
//
// Bound: latency.  A launch with one prefix per wave takes about 45 us, most of
// it the first pass over the code (9 KB per value of QB) and the chain of four
// layers; ten prefixes per wave, one after another with their keys and values
// from L2 where siblings share them, 80 us.  Loading the next prefixes' operands
// ahead (two sets of two to four) grew the code and the registers: 115 us.
// Against rows 0 .. s of every prefix evaluated again at every position (386 us
// a launch), 100,000 samples at K = 60 take 6.0 instead of 32.8 ms.
constexpr int kRowElems = 64;     // per layer and pair of heads: K [32], V [32]
constexpr int kCurLd = 40;        // LDS row of a prefix's current K or V (32 elements, padded)

struct RowsLds {
    TfLds<false> S;
    __bf16 cur[kTfWaves][2][16 * kCurLd];  // per wave: K and V of its prefixes' rows s
    int32_t path[kTfWaves][16][64];
};

template <int QB>
__device__ __forceinline__ void rows_tile(const Bf16View &M, const RowsArgs &A, RowsLds &R, int64_t tb, int cnt,
                                          const __bf16 *next_w, const float *next_v, int &vbuf) {
    typedef Op<false> OP;
    typedef bf16x8 Frag;
    TfLds<false> &S = R.S;
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c16 = l & 15, r0 = 4 * (l >> 4), kq = 8 * (l >> 4);
    const uint32_t half0 = l < 32 ? ~0u : 0u, half1 = ~half0;
    const int K = M.K, s = A.s, cq = s & 15;
    const float *wf = M.wf;
    const int64_t ent = (int64_t)M.L * 2 * kRowElems;  // elements of one prefix's row
    __bf16 *curK = R.cur[w][0], *curV = R.cur[w][1];
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // lane (c16, .): prefix tb + c16
    const bool own = c16 < cnt;
    const int64_t u = tb + (own ? c16 : 0);
    Key x{0ull, 0ull};
    if (own) {
        x.lo = A.keys[2 * u];
        x.hi = A.keys[2 * u + 1];
    }
    for (int p = 0; p < cnt; p++) R.path[w][p][l] = l < s ? A.path[(tb + p) * 64 + l] : 0;
    wave_sync();
    // the rows of key position 16 kb + c16, and which keys of the last block there are
    const __bf16 *base[QB + 1];
#pragma unroll
    for (int kb = 0; kb <= QB; kb++) base[kb] = A.rows.p[16 * kb + c16 < s ? 16 * kb + c16 : 0] + kq;
    const bool before = c16 < cq;
    const Frag none = {};
    // identity operands: head hs's 16 dims of a pair's 32
    Frag sel[2];
#pragma unroll
    for (int hs = 0; hs < 2; hs++)
#pragma unroll
        for (int e = 0; e < 8; e++) sel[hs][e] = (__bf16)(kq + e == 16 * hs + c16 ? 1.0f : 0.0f);
    Frag ones;
#pragma unroll
    for (int e = 0; e < 8; e++) ones[e] = (__bf16)1.0f;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    auto keep = [](bool mine, const f32x4 &v, f32x4 &to) {
#pragma unroll
        for (int i = 0; i < 4; i++) to[i] = mine ? v[i] : to[i];
    };

    f32x4 h[4];
    {
        const int o = K - s;  // orbital of the token before
        const int prev = s == 0 ? 4 : (int)key_bit(x, 2 * o) | ((int)key_bit(x, 2 * o + 1) << 1);
#pragma unroll
        for (int db = 0; db < 4; db++) {
            const int c = db * 16 + r0;
            h[db] = ld4(wf + M.fl.tok_emb + prev * kD + c) + ld4(wf + M.fl.pos_emb + s * kD + c);
        }
    }
    for (int layer = 0; layer < M.L; layer++) {
        const __bf16 *lw = M.wb + M.bl.layer0 + layer * M.bl.layer_stride;
        weights_ready();  // the attention half and the vectors are here; the last FFN is done
        load_half(S.wf, lw + kAttnElems, kFfnElems, w);
        const float *lv = S.vec[vbuf];
        if (cnt > 0) {
            Frag xn[2];
            normalize<false>(h, xn);
#pragma unroll
            for (int db = 0; db < 4; db++) h[db] += ld4(lv + kV_bo + db * 16 + r0);
#pragma unroll 1
            for (int hp = 0; hp < 2; hp++) {  // heads 2 hp, 2 hp + 1
                const int64_t at = ((int64_t)layer * 2 + hp) * kRowElems;
                Frag qh[2];
                {  // this row's K, V (kept for the positions after, and in LDS for this one) and Q
                    Quad2 k4[2], q4[2];
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        f32x4 qt = ld4(lv + kV_bqkv + 32 * hp + kq + 4 * t);
                        f32x4 kt = ld4(lv + kV_bqkv + 64 + 32 * hp + kq + 4 * t);
                        const float bv = lv[kV_bqkv + 128 + (2 * hp + t) * kDh + c16];
                        f32x4 v = f32x4{bv, bv, bv, bv};
#pragma unroll
                        for (int ks = 0; ks < 2; ks++) {
                            kt = OP::mma(wfrag<false>(S.wa, 2 * (4 + 2 * hp + t) + ks), xn[ks], kt);
                            v = OP::mma(xn[ks], wfrag<false>(S.wa, 2 * (8 + 2 * hp + t) + ks), v);
                            qt = OP::mma(wfrag<false>(S.wa, 2 * (2 * hp + t) + ks), xn[ks], qt);
                        }
                        k4[t] = Act<false>::pack(kt);
                        q4[t] = Act<false>::pack(qt);
#pragma unroll
                        for (int i = 0; i < 4; i++) curV[(r0 + i) * kCurLd + 16 * t + c16] = (__bf16)v[i];
                    }
                    const Frag kr = both(k4[0], k4[1]), qf = both(q4[0], q4[1]);
                    *reinterpret_cast<Frag *>(curK + c16 * kCurLd + kq) = kr;
                    qh[0] = half(qf, half0);
                    qh[1] = half(qf, half1);
                    wave_sync();
                    if (own) {
                        __bf16 *out = A.rows.p[s] + u * ent + at + kq;
                        *reinterpret_cast<Frag *>(out) = kr;
                        *reinterpret_cast<Frag *>(out + 32) = *reinterpret_cast<const Frag *>(curV + c16 * kCurLd + kq);
                    }
                }
                // one operand per key block of prefix p: lane = key 16 kb + c16, 8 of the pair's 32 columns
                auto fetch = [&](int p, int64_t off, const __bf16 *cur, Frag(&f)[QB + 1]) {
#pragma unroll
                    for (int kb = 0; kb < QB; kb++)
                        f[kb] = *reinterpret_cast<const Frag *>(base[kb] + R.path[w][p][16 * kb + c16] * ent + off);
                    const Frag now = *reinterpret_cast<const Frag *>(cur + p * kCurLd + kq);
                    f[QB] = c16 == cq ? now : none;
                    if (before)
                        f[QB] = *reinterpret_cast<const Frag *>(base[QB] + R.path[w][p][16 * QB + c16] * ent + off);
                };
                f32x4 st[2][QB + 1];
#pragma unroll
                for (int hs = 0; hs < 2; hs++)
#pragma unroll
                    for (int kb = 0; kb <= QB; kb++) st[hs][kb] = zero;
#pragma unroll 1
                for (int p = 0; p < cnt; p++) {
                    Frag kf[QB + 1];
                    fetch(p, at, curK, kf);
                    const bool mine = c16 == p;
#pragma unroll
                    for (int hs = 0; hs < 2; hs++)
#pragma unroll
                        for (int kb = 0; kb <= QB; kb++) keep(mine, mfma16(kf[kb], qh[hs], zero), st[hs][kb]);
                }
                Frag bp[2][2];
                f32x4 den[2];
#pragma unroll
                for (int hs = 0; hs < 2; hs++) {  // as in attend, query 16 QB + cq in every column
#pragma unroll
                    for (int i = 0; i < 4; i++) st[hs][QB][i] = r0 + i <= cq ? st[hs][QB][i] : -INFINITY;
                    float mx = -INFINITY;
#pragma unroll
                    for (int kb = 0; kb <= QB; kb++)
#pragma unroll
                        for (int i = 0; i < 4; i++) mx = __builtin_amdgcn_fmed3f(mx, st[hs][kb][i], INFINITY);  // the larger
                    mx = max_groups(mx);
                    Quad2 pq[4];
#pragma unroll
                    for (int kb = 0; kb < 4; kb++) {
                        pq[kb] = Quad2{{0u, 0u}};
                        if (kb <= QB) {
                            f32x4 e;
#pragma unroll
                            for (int i = 0; i < 4; i++) e[i] = __builtin_amdgcn_exp2f(st[hs][kb <= QB ? kb : 0][i] - mx);
                            pq[kb] = Act<false>::pack(e);
                        }
                    }
                    den[hs] = zero;
#pragma unroll
                    for (int pp = 0; 2 * pp <= QB; pp++) {
                        bp[hs][pp] = join(pq[2 * pp], pq[2 * pp + 1]);
                        den[hs] = mfma16(ones, bp[hs][pp], den[hs]);
                    }
                }
                f32x4 ot[2] = {zero, zero};
#pragma unroll 1
                for (int p = 0; p < cnt; p++) {
                    Frag vr[QB + 1];
                    fetch(p, at + 32, curV, vr);
                    const bool mine = c16 == p;
#pragma unroll
                    for (int hs = 0; hs < 2; hs++) {
                        Quad2 vq[4];
#pragma unroll
                        for (int kb = 0; kb < 4; kb++) {
                            vq[kb] = Quad2{{0u, 0u}};
                            if (kb <= QB) vq[kb] = Act<false>::pack(mfma16(vr[kb <= QB ? kb : 0], sel[hs], zero));
                        }
                        f32x4 o = zero;
#pragma unroll
                        for (int pp = 0; 2 * pp <= QB; pp++) o = mfma16(join(vq[2 * pp], vq[2 * pp + 1]), bp[hs][pp], o);
                        keep(mine, o, ot[hs]);
                    }
                }
                wave_sync();  // cur is read before the next pair rewrites it
                const Frag of = join(Act<false>::pack(ot[0] * __builtin_amdgcn_rcpf(den[0][0])),
                                     Act<false>::pack(ot[1] * __builtin_amdgcn_rcpf(den[1][0])));
#pragma unroll
                for (int db = 0; db < 4; db++) h[db] = OP::mma(wfrag<false>(S.wa, 24 + 2 * db + hp), of, h[db]);
            }
        }
        weights_ready();  // the FFN half is here; the attention half is consumed
        const bool last = layer + 1 == M.L;
        const __bf16 *nw = last ? next_w : lw + M.bl.layer_stride;
        const float *nv = last ? next_v : wf + M.fl.layer0 + (layer + 1) * M.fl.layer_stride;
        if (nw) {
            load_half(S.wa, nw, kAttnElems, w);
            load_half(S.vec[vbuf ^ 1], nv, kVecFloats, w);
        }
        vbuf ^= 1;
        if (cnt > 0) {
            Frag xn[2];
            normalize<false>(h, xn);
#pragma unroll 1
            for (int run = 0; run < 8; run++) {
                Quad2 gq[2];
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    f32x4 f = ld4(lv + kV_b1 + run * 32 + kq + 4 * t);
#pragma unroll
                    for (int ks = 0; ks < 2; ks++) f = OP::mma(wfrag<false>(S.wf, (2 * run + t) * 2 + ks), xn[ks], f);
                    f32x4 y;
#pragma unroll
                    for (int i = 0; i < 4; i++) y[i] = gelu_tab(S.gtab, f[i]);
                    gq[t] = Act<false>::pack(y);
                }
                const Frag g = both(gq[0], gq[1]);
#pragma unroll
                for (int db = 0; db < 4; db++) h[db] = OP::mma(wfrag<false>(S.wf, 32 + db * 8 + run), g, h[db]);
            }
#pragma unroll
            for (int db = 0; db < 4; db++) h[db] += ld4(lv + kV_b2 + db * 16 + r0);
        }
    }
    if (cnt <= 0) return;
    // final LayerNorm, head, mask and the four conditionals, in lanes 0..15
    float rstd, sh, z[4] = {0.f, 0.f, 0.f, 0.f};
    row_stats(h, rstd, sh);
#pragma unroll
    for (int db = 0; db < 4; db++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const f32x4 hw4 = ld4(wf + M.fl.head_w + (db * 16 + r0 + i) * 4);
            const float y = fmaf(h[db][i], rstd, sh);
#pragma unroll
            for (int t = 0; t < 4; t++) z[t] = fmaf(y, hw4[t], z[t]);
        }
#pragma unroll
    for (int t = 0; t < 4; t++) z[t] = sum_groups(z[t]);
    if (l < 16 && own) {
        const uint64_t even = 0x5555555555555555ull;
        const int up = __popcll(x.lo & even) + __popcll(x.hi & even);
        const int dn = __popcll(x.lo & ~even) + __popcll(x.hi & ~even);
        const int rem = K - 1 - s, orb = K - 1 - s;
        float mx = -INFINITY;
        bool ok[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            z[t] += wf[M.fl.head_b + t] + wf[M.fl.bias + orb * 4 + t];
            const int bu = t & 1, bd = t >> 1;
            ok[t] = (up + bu <= M.n_up) && (dn + bd <= M.n_dn) && (M.n_up - up - bu <= rem) && (M.n_dn - dn - bd <= rem);
            if (ok[t]) mx = fmaxf(mx, z[t]);
        }
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < 4; t++)
            if (ok[t]) sum += __expf(z[t] - mx);
        const float lden = __logf(sum);
#pragma unroll
        for (int t = 0; t < 4; t++) A.cond[u * 4 + t] = ok[t] ? (double)((z[t] - mx) - lden) : -INFINITY;
    }
}

// A tile holds kTfWaves x A.per prefixes; the blocks share the tiles as in
// transformer().
__global__ void __launch_bounds__(64 * kTfWaves) k_transformer_rows(Bf16View M, RowsArgs A) {
    __shared__ __align__(16) RowsLds R;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i = threadIdx.x; i < kGeluN; i += blockDim.x)
        R.S.gtab[i] = make_float2(M.wf[M.fl.gelu + 2 * i], M.wf[M.fl.gelu + 2 * i + 1]);
    const int64_t per_tile = (int64_t)kTfWaves * A.per, T = (A.n + per_tile - 1) / per_tile;
    const __bf16 *w0 = M.wb + M.bl.layer0;
    const float *v0 = M.wf + M.fl.layer0;
    if ((int64_t)blockIdx.x >= T) return;
    int vbuf = 0;
    load_half(R.S.wa, w0, kAttnElems, w);
    load_half(R.S.vec[0], v0, kVecFloats, w);
    for (int64_t tile = blockIdx.x; tile < T; tile += gridDim.x) {
        const int64_t tb = tile * per_tile + (int64_t)w * A.per, left = A.n - tb;
        const int cnt = __builtin_amdgcn_readfirstlane((int)(left < 0 ? 0 : left < A.per ? left : A.per));
        const __bf16 *next_w = tile + gridDim.x < T ? w0 : nullptr;
        switch (A.s >> 4) {
            case 0: rows_tile<0>(M, A, R, tb, cnt, next_w, v0, vbuf); break;
            case 1: rows_tile<1>(M, A, R, tb, cnt, next_w, v0, vbuf); break;
            case 2: rows_tile<2>(M, A, R, tb, cnt, next_w, v0, vbuf); break;
            default: rows_tile<3>(M, A, R, tb, cnt, next_w, v0, vbuf); break;
        }
    }
}

nnqs_status tf_launch_rows(int cus, hipStream_t st, const Bf16View &M, RowsArgs A) {
    // as many prefixes per wave as give every CU's waves some, 16 at most
    const int64_t waves = (int64_t)cus * kTfWaves;
    A.per = (int)std::min<int64_t>(16, (A.n + waves - 1) / waves);
    const int64_t per_tile = (int64_t)kTfWaves * A.per, T = (A.n + per_tile - 1) / per_tile;
    hipLaunchKernelGGL(k_transformer_rows, dim3((unsigned)std::min<int64_t>(T, cus)), dim3(64 * kTfWaves), 0,
                       st, M, A);
    NNQS_HIP_CHECK(hipGetLastError());
    return NNQS_OK;
}

size_t rows_entry_bytes(int n_layers) { return (size_t)n_layers * 2 * kRowElems * sizeof(__bf16); }

}  // namespace nnqs
