// Batch autoregressive sampling (paper: Section 3.1) on the device: the
// samples of one VMC iteration are drawn together by following the unique
// prefixes of the autoregressive ansatz with their weights.  At sequence
// position s every unique prefix u (weight c_u) gets its conditional
// pi(t | prefix) from the network (the Eq. 12 mask included), each of its
// c_u sample slots draws one token from a counter-based generator, which
// splits c_u multinomially among the four children, and children with zero
// weight are dropped.  After K positions the prefixes are the unique samples
// and their weights the occurrence counts.
//
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC 2011),
// counter (slot mod 2^32, slot / 2^32, s, 0x42415300), key = the seed, the
// top 53 bits of the first two output words; slots are numbered in prefix
// order, children are kept in (parent, token) order, so the result depends
// only on the seed and the conditionals.
#include <algorithm>
#include <atomic>
#include <cmath>

#include "transformer.hpp"

namespace nnqs {

__device__ __forceinline__ double bas_uniform(uint64_t seed, int s, uint64_t i) {
    uint32_t c0 = (uint32_t)i, c1 = (uint32_t)(i >> 32), c2 = (uint32_t)s, c3 = 0x42415300u;
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int r = 0; r < 10; r++) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n1 = (uint32_t)p1;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1, n3 = (uint32_t)p0;
        c0 = n0;
        c1 = n1;
        c2 = n2;
        c3 = n3;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    const uint64_t x = ((uint64_t)c0 << 32) | c1;
    return (double)(x >> 11) * (1.0 / 9007199254740992.0);
}

// Token of a slot: the allowed tokens in order 0..3, probabilities summed
// until the running sum exceeds u (the last allowed one if rounding leaves u
// above the total).
__device__ __forceinline__ int bas_token(const double *logp, double u) {
    double acc = 0.0;
    int last = -1;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        if (!(logp[t] > -INFINITY)) continue;
        last = t;
        acc += exp(logp[t]);
        if (u < acc) return t;
    }
    return last;
}

// One token per sample slot i < total; slot i belongs to the prefix u with
// offs[u] <= i < offs[u + 1].  A block takes 256 slots in a row: its threads
// together find the first one's prefix (256 marks per round), and as every
// prefix has a slot, the block's prefixes are the next 256 at most, whose
// offsets go through LDS and its draws are counted there: one atomic per
// (prefix, token) of a block.
__global__ void __launch_bounds__(256) k_bas_draw(uint64_t total, int s, uint64_t seed,
                                                  const uint64_t *__restrict__ offs, int64_t n,
                                                  const double *__restrict__ cond,
                                                  unsigned long long *__restrict__ child) {
    __shared__ uint64_t so[256];
    __shared__ uint32_t drawn[4 * 256];
    const int t = threadIdx.x;
    for (uint64_t base = (uint64_t)blockIdx.x * 256; base < total; base += (uint64_t)gridDim.x * 256) {
        int64_t lo = 0, hi = n;  // offs[lo] <= base, and offs[hi] > base or hi = n
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + 255) / 256, q = lo + t * step;
            const int c = __syncthreads_count(q < hi && offs[q] <= base);
            lo += (c - 1) * step;
            hi = lo + step < hi ? lo + step : hi;
        }
        so[t] = lo + t < n ? offs[lo + t] : ~0ull;
#pragma unroll
        for (int q = 0; q < 4; q++) drawn[t + 256 * q] = 0;
        __syncthreads();
        const uint64_t i = base + t;
        if (i < total) {
            int k = 0;
#pragma unroll
            for (int step = 128; step >= 1; step >>= 1)
                if (so[k + step] <= i) k += step;
            const int64_t u = lo + k;
            const int tok = bas_token(cond + 4 * u, bas_uniform(seed, s, i));
            // no allowed token: the prefix leaves the sector (not for valid models)
            if (tok >= 0) atomicAdd(&drawn[4 * k + tok], 1u);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const uint32_t c = drawn[t + 256 * q];
            if (c) atomicAdd(child + 4 * lo + t + 256 * q, (unsigned long long)c);
        }
        __syncthreads();  // so and drawn are read before the next slots' are set
    }
}

constexpr int kBasBlock = 256;  // prefixes per block of the two kernels below

__device__ __forceinline__ int children(const unsigned long long *child, int64_t u) {
    return (child[4 * u] > 0) + (child[4 * u + 1] > 0) + (child[4 * u + 2] > 0) + (child[4 * u + 3] > 0);
}

// Sum over the block of v, for every thread (sh: 4 values).
__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t *sh) {
    for (int d = 32; d; d >>= 1) v += __shfl_xor(v, d, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

__device__ __forceinline__ int64_t slots(const unsigned long long *child, int64_t u) {
    return (int64_t)((child[4 * u] + child[4 * u + 1]) + (child[4 * u + 2] + child[4 * u + 3]));
}

// Children of each block's prefixes, and the slots they hold.
__global__ void __launch_bounds__(kBasBlock) k_bas_count(int64_t n, const unsigned long long *__restrict__ child,
                                                         int64_t *__restrict__ blk) {
    __shared__ int64_t sh[4];
    const int64_t u = (int64_t)blockIdx.x * kBasBlock + threadIdx.x;
    const int64_t c = block_sum(u < n ? children(child, u) : 0, sh);
    const int64_t s = block_sum(u < n ? slots(child, u) : 0, sh);
    if (threadIdx.x == 0) {
        blk[2 * (int64_t)blockIdx.x] = c;
        blk[2 * (int64_t)blockIdx.x + 1] = s;
    }
}

// The arrays of one position's prefixes.
struct BasLevel {
    uint64_t *keys, *cnt, *offs;  // key, slots, first slot
    double *lp;                   // log-probability of the path
    unsigned long long *child;    // [4] slots drawn for each token
    int32_t *path;                // [64] ancestors by position (with cached rows; else null)
};

// Children of prefix u, in (parent, token) order: the parent's key with the
// token of position s (spatial orbital K-1-s: up bit 2i, down bit 2i+1), its
// slots, the path's log-probability and ancestors.  A block's first child
// follows the children of the blocks before it; every block adds those up
// itself (a scan by one block and a launch of its own per array took 52 us a
// position, of which 1,024 additions in a row were most).  No child beyond
// `cap` is written; the last block reports the total.
__global__ void __launch_bounds__(kBasBlock) k_bas_expand(int64_t n, int64_t cap, int K, int s, BasLevel P, BasLevel N,
                                                          const double *__restrict__ cond,
                                                          const int64_t *__restrict__ blk, int64_t *__restrict__ total) {
    __shared__ int64_t sh[4];
    __shared__ int wsum[4];
    __shared__ int64_t wslots[4];
    __shared__ uint8_t parent[4 * kBasBlock];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int64_t before = 0, off = 0;  // children and slots of the blocks before
    for (int64_t b = t; b < (int64_t)blockIdx.x; b += kBasBlock) {
        before += blk[2 * b];
        off += blk[2 * b + 1];
    }
    before = block_sum(before, sh);
    off = block_sum(off, sh);
    const int64_t u = (int64_t)blockIdx.x * kBasBlock + t;
    const int mine = u < n ? children(P.child, u) : 0;
    const int64_t held = u < n ? slots(P.child, u) : 0;
    int pos = mine;  // inclusive scans over the wave
    int64_t sl = held;
    for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(pos, d, 64);
        const int64_t x = __shfl_up(sl, d, 64);
        if (lane >= d) {
            pos += v;
            sl += x;
        }
    }
    if (lane == 63) {
        wsum[w] = pos;
        wslots[w] = sl;
    }
    __syncthreads();
    pos -= mine;
    off += sl - held;
    for (int q = 0; q < w; q++) {
        pos += wsum[q];
        off += wslots[q];
    }
    const int all = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (blockIdx.x == gridDim.x - 1 && t == 0) *total = before + all;
    if (u < n) {
        const int i = K - 1 - s;
        for (int tk = 0; tk < 4; tk++) {
            const unsigned long long c = P.child[4 * u + tk];
            if (!c) continue;
            const int64_t p = before + pos;
            parent[pos++] = (uint8_t)t;
            if (p < cap) {
                Key x;
                x.lo = P.keys[2 * u];
                x.hi = P.keys[2 * u + 1];
                if (tk & 1) key_flip(x, 2 * i);
                if (tk & 2) key_flip(x, 2 * i + 1);
                N.keys[2 * p] = x.lo;
                N.keys[2 * p + 1] = x.hi;
                N.cnt[p] = c;
                N.offs[p] = (uint64_t)off;
                N.lp[p] = P.lp[u] + cond[4 * u + tk];
#pragma unroll
                for (int q = 0; q < 4; q++) N.child[4 * p + q] = 0;
            }
            off += (int64_t)c;
        }
    }
    if (!N.path) return;
    __syncthreads();
    const int q0 = 4 * (t & 15);  // 16 lanes per child, four positions each
    if (q0 > s) return;
#pragma unroll 4
    for (int j = t >> 4; j < all; j += kBasBlock / 16) {
        const int64_t p = before + j, up = (int64_t)blockIdx.x * kBasBlock + parent[j];
        int4 v = q0 < s ? *reinterpret_cast<const int4 *>(P.path + up * 64 + q0) : int4{0, 0, 0, 0};
        if (q0 == s) v.x = (int32_t)up;
        else if (q0 + 1 == s) v.y = (int32_t)up;
        else if (q0 + 2 == s) v.z = (int32_t)up;
        else if (q0 + 3 == s) v.w = (int32_t)up;
        if (p < cap) *reinterpret_cast<int4 *>(N.path + p * 64 + q0) = v;
    }
}

__global__ void k_bas_finish(int64_t n, const uint64_t *__restrict__ cnt, const double *__restrict__ lp,
                             uint32_t *__restrict__ counts_out, double *__restrict__ logabs_out) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    counts_out[u] = (uint32_t)cnt[u];
    logabs_out[u] = 0.5 * lp[u];
}

__global__ void k_bas_init(BasLevel P, uint64_t total) {
    P.keys[0] = 0ull;
    P.keys[1] = 0ull;
    P.cnt[0] = total;
    P.offs[0] = 0ull;
    P.lp[0] = 0.0;
    for (int q = 0; q < 4; q++) P.child[q] = 0;
}

}  // namespace nnqs

// Workspace of a sampling call: two levels of prefixes, scratch of one level,
// and for the BF16 network each level's paths and every position's rows, all
// grown to the number of prefixes seen.  A call takes the model's workspace, or
// makes one where another call has it, and leaves it with the model if it holds
// at most kBasKeep bytes and those of all models at most twice as many (a call
// that finds none takes 1.3 ms longer at K = 60 and 100,000 samples).
struct BasWork {
    size_t level_cap[2] = {}, path_cap[2] = {}, scratch_cap = 0, row_bytes[64] = {};
    void *level[2] = {}, *path[2] = {};
    double *cond = nullptr, *la = nullptr;
    int64_t *blk = nullptr, *total = nullptr;  // total: host memory
    void *rows[64] = {};
    size_t bytes() const {
        size_t b = 40 * scratch_cap;
        for (int i = 0; i < 2; i++) b += 72 * level_cap[i] + 256 * path_cap[i];
        for (size_t r : row_bytes) b += r;
        return b;
    }
    ~BasWork() {
        for (int i = 0; i < 2; i++) {
            (void)hipFree(level[i]);
            (void)hipFree(path[i]);
        }
        (void)hipFree(cond);
        (void)hipFree(la);
        (void)hipFree(blk);
        (void)hipHostFree(total);
        for (void *r : rows) (void)hipFree(r);
    }
};

namespace nnqs {

constexpr size_t kBasKeep = (size_t)4 << 30;
static std::atomic<size_t> g_bas_kept{0};  // held by models between their calls

// The model's idle workspace, which its next owner takes off the sum.
static BasWork *bas_take(nnqs_model *m) {
    BasWork *w = m->bas_work.exchange(nullptr);
    if (w) g_bas_kept -= w->bytes();
    return w;
}

void bas_model_free(nnqs_model *m) { delete bas_take(m); }

// Holds a workspace for one call; the stream is idle when it goes back.
struct BasHold {
    nnqs_model *m;
    hipStream_t st;
    BasWork *w;
    bool drop = false;  // give its memory back
    BasHold(nnqs_model *model, hipStream_t stream) : m(model), st(stream), w(bas_take(model)) {
        if (!w) w = new BasWork();
    }
    ~BasHold() {
        (void)hipStreamSynchronize(st);
        const size_t b = w->bytes();
        size_t kept = g_bas_kept.load();
        while (!drop && b <= kBasKeep && kept + b <= 2 * kBasKeep)
            if (g_bas_kept.compare_exchange_weak(kept, kept + b)) {
                BasWork *none = nullptr;
                if (m->bas_work.compare_exchange_strong(none, w)) return;
                g_bas_kept -= b;  // another call has left one
                break;
            }
        delete w;
    }
};

static bool bas_alloc(void **p, size_t bytes) {
    (void)hipFree(*p);
    *p = nullptr;
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    *p = nullptr;
    return false;
}

// Entries to allocate for `need` of at most `most`: twice as many and no fewer
// than 2^17 (45 MB of a level with its paths), so that a call grows its arrays a
// few times only; each time costs some 0.2 ms.
static size_t bas_want(size_t need, size_t most) { return std::min(std::max(2 * need, (size_t)1 << 17), most); }

// Room for n prefixes in level i, and for the scratch of a level of n; what was
// in them is not kept.
static bool bas_room(BasWork &W, int i, size_t n, size_t most) {
    if (W.level_cap[i] >= n) return true;
    const size_t cap = bas_want(n, most);
    W.level_cap[i] = 0;
    if (!bas_alloc(&W.level[i], cap * 72)) return false;
    W.level_cap[i] = cap;
    return true;
}

static bool bas_scratch(BasWork &W, size_t n, size_t most) {
    if (!W.total && hipHostMalloc(reinterpret_cast<void **>(&W.total), 8) != hipSuccess) {
        (void)hipGetLastError();
        W.total = nullptr;
        return false;
    }
    if (W.scratch_cap >= n) return true;
    const size_t cap = bas_want(n, most);
    W.scratch_cap = 0;
    if (!bas_alloc(reinterpret_cast<void **>(&W.cond), cap * 32) || !bas_alloc(reinterpret_cast<void **>(&W.la), cap * 8) ||
        !bas_alloc(reinterpret_cast<void **>(&W.blk), (cap / kBasBlock + 1) * 16))
        return false;
    W.scratch_cap = cap;
    return true;
}

// Memory for `bytes` more, a quarter of what is free at a time at most.
static bool bas_spare(size_t bytes) {
    size_t free_b = 0, all_b = 0;
    return hipMemGetInfo(&free_b, &all_b) == hipSuccess && bytes <= free_b / 4;
}

static bool bas_paths(BasWork &W, int i, size_t n) {
    if (W.path_cap[i] >= n) return true;
    const size_t cap = W.level_cap[i];
    if (!bas_spare(cap * 256)) return false;
    W.path_cap[i] = 0;
    if (!bas_alloc(&W.path[i], cap * 256)) return false;
    W.path_cap[i] = cap;
    return true;
}

static BasLevel bas_level(const BasWork &W, int i, bool paths) {
    BasLevel v{};
    const size_t cap = W.level_cap[i];
    uint8_t *p = static_cast<uint8_t *>(W.level[i]);
    v.keys = reinterpret_cast<uint64_t *>(p);
    v.cnt = reinterpret_cast<uint64_t *>(p + cap * 16);
    v.offs = reinterpret_cast<uint64_t *>(p + cap * 24);
    v.lp = reinterpret_cast<double *>(p + cap * 32);
    v.child = reinterpret_cast<unsigned long long *>(p + cap * 40);
    v.path = paths ? static_cast<int32_t *>(W.path[i]) : nullptr;
    return v;
}

// Room for `need` bytes of rows at position s, with a quarter to spare; false:
// not to be had.
static bool bas_rows(BasWork &W, int s, size_t need, size_t most) {
    if (W.row_bytes[s] >= need) return true;
    const size_t want = std::min(need + need / 4, most);
    if (!bas_spare(want)) return false;
    W.row_bytes[s] = 0;
    if (!bas_alloc(&W.rows[s], want)) return false;
    W.row_bytes[s] = want;
    return true;
}

}  // namespace nnqs

using namespace nnqs;

extern "C" nnqs_status nnqs_bas(nnqs_model *model, int32_t precision, uint64_t seed, uint64_t n_samples,
                                int64_t capacity, uint64_t *keys_out, uint32_t *counts_out, double *logabs_out,
                                double *phase_out, int64_t *n_unique, void *stream) {
    clear_error();
    if (!model || !keys_out || !counts_out || !logabs_out || !n_unique) return fail(NNQS_EINVAL, "null pointer argument");
    if (n_samples < 1 || n_samples > 0xFFFFFFFFull) return fail(NNQS_EINVAL, "n_samples must be in [1, 2^32 - 1]");
    if (capacity < 1) return fail(NNQS_EINVAL, "capacity must be positive");
    if (precision == NNQS_FP64 && !f64_shape_ok(model->desc))
        return fail(NNQS_EUNSUPPORTED, "FP64 sampling needs d_model 64 and 4 heads");
    if (precision == NNQS_BF16 && !model->bf16_ok) return fail(NNQS_EUNSUPPORTED, "model shape has no BF16 path");
    if (precision != NNQS_FP64 && precision != NNQS_BF16) return fail(NNQS_EUNSUPPORTED, "sampling runs in FP64 or BF16");
    hipStream_t st = as_stream(stream);
    const int K = model->desc.n_orb;
    const bool bf16 = precision == NNQS_BF16;
    // every prefix has a slot: never more prefixes than samples
    const size_t cap = (size_t)std::min<uint64_t>((uint64_t)capacity, n_samples);
    BasHold hold(model, st);
    BasWork &W = *hold.w;
    const auto no_memory = [&](int64_t prefixes) {
        hold.drop = true;
        return fail(NNQS_ENOMEM, "sampling scratch for %lld prefixes", (long long)prefixes);
    };
    bool cached = bf16;  // rows of the positions before kept
    const size_t entry = rows_entry_bytes(model->desc.n_layers);
    int at = 0;  // level of the prefixes
    if (!bas_room(W, at, 1, cap)) return no_memory(1);
    BasLevel P = bas_level(W, at, false);
    hipLaunchKernelGGL(k_bas_init, dim3(1), dim3(1), 0, st, P, (uint64_t)n_samples);
    const unsigned dg = (unsigned)std::min<uint64_t>((n_samples + 255) / 256, 8192);
    int64_t n = 1;
    for (int s = 0; s < K; s++) {
        const size_t next = std::min((size_t)(4 * n), cap);  // children, at most
        if (!bas_scratch(W, (size_t)n, cap) || !bas_room(W, at ^ 1, next, cap)) return no_memory((int64_t)next);
        cached = cached && bas_paths(W, at ^ 1, next) && bas_rows(W, s, (size_t)n * entry, cap * entry);
        BasLevel N = bas_level(W, at ^ 1, cached);
        if (!cached) P.path = nullptr;
        nnqs_status r;
        if (cached) {
            RowsArgs A{};
            A.keys = P.keys;
            A.path = P.path;
            A.n = n;
            A.s = s;
            A.cond = W.cond;
            for (int i = 0; i <= s; i++) A.rows.p[i] = static_cast<__bf16 *>(W.rows[i]);
            r = enqueue_bf16_rows(model, A, st);
        } else {
            r = bf16 ? enqueue_bf16_cond(model, P.keys, n, s, W.cond, W.la, st)
                     : enqueue_logpsi_f64(model, P.keys, n, W.la, nullptr, st, s, W.cond);
        }
        if (r != NNQS_OK) return r;
        hipLaunchKernelGGL(k_bas_draw, dim3(dg), dim3(256), 0, st, (uint64_t)n_samples, s, seed,
                           (const uint64_t *)P.offs, n, (const double *)W.cond, P.child);
        const unsigned nb = (unsigned)((n + kBasBlock - 1) / kBasBlock);
        hipLaunchKernelGGL(k_bas_count, dim3(nb), dim3(kBasBlock), 0, st, n, (const unsigned long long *)P.child, W.blk);
        hipLaunchKernelGGL(k_bas_expand, dim3(nb), dim3(kBasBlock), 0, st, n, (int64_t)cap, K, s, P, N,
                           (const double *)W.cond, (const int64_t *)W.blk, W.total);
        NNQS_HIP_CHECK(hipGetLastError());
        NNQS_HIP_CHECK(hipStreamSynchronize(st));
        const int64_t m = *const_cast<volatile int64_t *>(W.total);
        if (m > (int64_t)cap) return fail(NNQS_ERANGE, "%lld prefixes at position %d exceed the capacity %lld",
                                          (long long)m, s, (long long)capacity);
        if (m < 1) return fail(NNQS_EHIP, "no token is allowed at position %d", s);
        P = N;
        at ^= 1;
        n = m;
    }
    NNQS_HIP_CHECK(hipMemcpyAsync(keys_out, P.keys, (size_t)n * 16, hipMemcpyDeviceToDevice, st));
    hipLaunchKernelGGL(k_bas_finish, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, (const uint64_t *)P.cnt,
                       (const double *)P.lp, counts_out, logabs_out);
    NNQS_HIP_CHECK(hipGetLastError());
    if (phase_out) {
        if (!bf16 && !bas_scratch(W, (size_t)n, cap)) return no_memory(n);
        nnqs_status r = bf16 ? enqueue_phase_bf16(model, keys_out, n, phase_out, st)
                             : enqueue_logpsi(model, keys_out, n, precision, W.la, phase_out, st);
        if (r != NNQS_OK) return r;
    }
    NNQS_HIP_CHECK(hipStreamSynchronize(st));
    *n_unique = n;
    return NNQS_OK;
}
