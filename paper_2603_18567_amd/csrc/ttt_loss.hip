// In-place backward of the log-softmax loss (Sec. 4.2.2, Alg. 3) for gfx950: one workgroup per row, bound by
// HBM.  A row is read ONCE -- logits and target -- and kept on the compute unit until the gradient is
// written, so the HBM traffic is the algorithmic 3 * V * element size per row:
//   ttt_loss_bwd_kernel       up to 8 sixteen-byte vectors of each per thread, in registers: rows of 8192 fp32 or
//                             16384 bf16 values with 256 threads, of four times as many (the draft
//                             vocabularies) with 1024
//   ttt_loss_bwd_long_kernel  longer rows: 512 threads keep up to 26 vectors of each in registers and 9 in LDS
//                             (71680 fp32 or 143360 bf16 values); only what is beyond that is read twice
// A row may start at any element (a contiguous tensor with a ragged vocabulary has such rows): its vectors start
// at the first 16-byte boundary of the logits, the few columns before it are single elements of the first
// threads.  Vectors are loaded with the alignment of one element all the same (the hardware takes any), which
// the target's rows need where they lie differently.  (8192 x 4096 bf16 119 -> 35 us and 4096 x 50257 bf16 666 ->
// 274 with the smaller workgroups, the vectors on ragged rows, and all loads of a row requested before the first
// is used.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/ttt_attn.h"
#include "../../include/ttt_loss.h"
#include "ttt_args.hpp"

namespace ttt {

constexpr int kCacheIters = 8;
constexpr float kLog2eL = 1.44269504088896340736f;

template <typename T> struct LossVec;
template <> struct LossVec<float> {
    static constexpr int N = 4;
    typedef f32x4 raw;
    typedef f32x4 mem __attribute__((aligned(4)));
    TTT_DEV static void unpack(const raw& r, float (&o)[N]) {
#pragma unroll
        for (int i = 0; i < N; ++i) o[i] = r[i];
    }
    TTT_DEV static raw pack(const float (&o)[N]) { return raw{o[0], o[1], o[2], o[3]}; }
};
template <> struct LossVec<__bf16> {
    static constexpr int N = 8;
    typedef bf16x8 raw;
    typedef bf16x8 mem __attribute__((aligned(2)));
    TTT_DEV static void unpack(const raw& r, float (&o)[N]) {
#pragma unroll
        for (int i = 0; i < N; ++i) o[i] = (float)r[i];
    }
    TTT_DEV static raw pack(const float (&o)[N]) {
        raw r;
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = (__bf16)o[i];
        return r;
    }
};

// columns [c0, c0 + N) of a row: a whole vector, and one that may reach past the row's end (columns there read as
// `fill`).  NT: the accesses are marked as not to be kept by the caches (see the rule in launch_loss_t).
template <typename T, bool NT> TTT_DEV typename LossVec<T>::raw load_vec(const T* row, int c0) {
    const auto* at = reinterpret_cast<const typename LossVec<T>::mem*>(row + c0);
    if constexpr (NT) return __builtin_nontemporal_load(at);
    else return *at;
}
template <typename T, bool NT> TTT_DEV void store_vec(T* row, int c0, const typename LossVec<T>::raw& v) {
    auto* at = reinterpret_cast<typename LossVec<T>::mem*>(row + c0);
    if constexpr (NT) __builtin_nontemporal_store(v, at);
    else *at = v;
}
template <typename T, bool NT> TTT_DEV typename LossVec<T>::raw load_edge(const T* row, int c0, int vocab, float fill) {
    constexpr int N = LossVec<T>::N;
    if (c0 + N <= vocab) return load_vec<T, NT>(row, c0);
    float o[N];
#pragma unroll
    for (int e = 0; e < N; ++e) o[e] = c0 + e < vocab ? (float)row[c0 + e] : fill;
    return LossVec<T>::pack(o);
}
template <typename T, bool NT> TTT_DEV void store_edge(T* row, int c0, int vocab, const typename LossVec<T>::raw& v) {
    constexpr int N = LossVec<T>::N;
    if (c0 + N <= vocab) {
        store_vec<T, NT>(row, c0, v);
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (c0 + e < vocab) row[c0 + e] = v[e];
    }
}
// columns of a row before its first 16-byte boundary (at most vocab of them)
template <typename T> TTT_DEV int columns_before_boundary(const T* row, int vocab) {
    const int n = (int)((16 - (reinterpret_cast<uintptr_t>(row) & 15)) & 15) / (int)sizeof(T);
    return n < vocab ? n : vocab;
}
// the gradient of one vector: pi * s = exp(z - max) * (s / sum), minus p * g
template <typename T>
TTT_DEV typename LossVec<T>::raw loss_grad(const typename LossVec<T>::raw& zr, const typename LossVec<T>::raw& pr, float mc, float w, float g) {
    constexpr int N = LossVec<T>::N;
    float zv[N], pv[N], o[N];
    LossVec<T>::unpack(zr, zv);
    LossVec<T>::unpack(pr, pv);
#pragma unroll
    for (int e = 0; e < N; ++e) o[e] = fmaf(fast_exp2(fmaf(zv[e], kLog2eL, -mc)), w, -pv[e] * g);
    return LossVec<T>::pack(o);
}

// workgroup-wide reductions: wave butterflies, then one LDS round
TTT_DEV float wave_max(float v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v = fmaxf(v, __shfl_xor(v, s, 64));
    return v;
}
TTT_DEV float wave_sum(float v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, 64);
    return v;
}
template <int WAVES, bool MAX> TTT_DEV float block_reduce(float v, float (&red)[WAVES]) {
    v = MAX ? wave_max(v) : wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) v = MAX ? fmaxf(v, red[w]) : v + red[w];
    return v;
}

// What the first sweep over a row collects, with a running maximum so that the exponentials are done as the loads
// arrive.  mk: the maximum times log2(e), rounded -- what the exponents are taken against, here and in the end, so
// that its rounding (2^-24 |mk|) cancels between the terms and their sum; l: the sum of 2^(z log2(e) - mk).
template <typename T> struct LossSums {
    float mk = -INFINITY, l = 0.f, sp = 0.f;
    TTT_DEV void take(const typename LossVec<T>::raw& zr, const typename LossVec<T>::raw& pr) {
        constexpr int N = LossVec<T>::N;
        float zv[N], pv[N];
        LossVec<T>::unpack(zr, zv);
        LossVec<T>::unpack(pr, pv);
        float mx = zv[0];
#pragma unroll
        for (int e = 1; e < N; ++e) mx = fmaxf(mx, zv[e]);
        mx = fmaxf(mk, mx * kLog2eL);
        const float off = mx == -INFINITY ? 0.f : mx;
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            sum += fast_exp2(fmaf(zv[e], kLog2eL, -off));
            sp += pv[e];
        }
        l = fmaf(l, fast_exp2(mk - off), sum);
        mk = mx;
    }
    TTT_DEV void take_one(float z, float p) {
        const float mx = fmaxf(mk, z * kLog2eL);
        const float off = mx == -INFINITY ? 0.f : mx;
        l = fmaf(l, fast_exp2(mk - off), fast_exp2(fmaf(z, kLog2eL, -off)));
        sp += p;
        mk = mx;
    }
    // over the workgroup: the row's maximum and the factor of its exponentials, g * sum(p) / sum(exp)
    template <int WAVES> TTT_DEV void finish(float (&red)[3][WAVES], float g, float& mc, float& w) {
        sp = wave_sum(sp);
        if ((threadIdx.x & 63) == 0) red[1][threadIdx.x >> 6] = sp;
        mc = block_reduce<WAVES, true>(mk, red[0]);
        float sum_p = red[1][0];
#pragma unroll
        for (int i = 1; i < WAVES; ++i) sum_p += red[1][i];
        l *= mk == -INFINITY ? 0.f : fast_exp2(mk - mc);
        w = g * sum_p / block_reduce<WAVES, false>(l, red[2]);
    }
};

// One row: element e of this thread's vector number `it` is column ((it * THREADS + tid) * N + e).
template <typename T, int THREADS, bool NT>
__global__ __launch_bounds__(THREADS) void ttt_loss_bwd_kernel(T* __restrict__ logits, const T* __restrict__ target,
                                                               const float* __restrict__ grad, int vocab,
                                                               int64_t z_stride, int64_t p_stride) {
    using LV = LossVec<T>;
    constexpr int N = LV::N;
    __shared__ float red[3][THREADS / 64];
    const int tid = threadIdx.x;
    const int64_t row = blockIdx.x;
    T* z = logits + row * z_stride;
    const T* p = target + row * p_stride;
    const float g = grad[row];
    const int n_head = columns_before_boundary(z, vocab);
    z += n_head;
    p += n_head;
    vocab -= n_head;
    const int n_iter = (vocab + N * THREADS - 1) / (N * THREADS);   // at most kCacheIters: the launcher sees to it
    auto col = [&](int it) { return (it * THREADS + tid) * N; };

    typename LV::raw zc[kCacheIters], pc[kCacheIters];
#pragma unroll
    for (int it = 0; it < kCacheIters; ++it)
        if (it < n_iter) {
            zc[it] = load_edge<T, NT>(z, col(it), vocab, -INFINITY);
            pc[it] = load_edge<T, NT>(p, col(it), vocab, 0.f);
        }
    LossSums<T> sums;
#pragma unroll
    for (int it = 0; it < kCacheIters; ++it)
        if (it < n_iter) sums.take(zc[it], pc[it]);
    if (tid < n_head) sums.take_one((float)z[tid - n_head], (float)p[tid - n_head]);
    float mc, w;
    sums.template finish<THREADS / 64>(red, g, mc, w);
    if (tid < n_head)
        z[tid - n_head] = (T)fmaf(fast_exp2(fmaf((float)z[tid - n_head], kLog2eL, -mc)), w, -(float)p[tid - n_head] * g);
#pragma unroll
    for (int it = 0; it < kCacheIters; ++it)
        if (it < n_iter) store_edge<T, NT>(z, col(it), vocab, loss_grad<T>(zc[it], pc[it], mc, w, g));
}

// A row that registers alone do not hold: slabs of 512 vectors, the first NREG of them in registers, the next
// kLdsSlabs in LDS (each thread reads back what it wrote), and the rest, read again from memory; columns past
// the last whole slab are one more vector per thread.  The first sweep works with a running maximum, so that
// its exponentials are done while the next loads are in flight and one pair of reductions ends it.  Slabs that
// are read twice come first and last, when the registers are free for loads in flight, and are the only ones that
// the caches are asked to keep.  512 threads rather than 1024: the 256 registers of each hold more of the row
// beside the working values.  Measured against two full reads of the row: 4096 x 151936 bf16 1153 -> 696 us
// (5.4 TB/s of the algorithmic bytes; a device copy reaches 5.2), fp32 2448 -> 1515, 2048 x 65543 bf16 600 -> 166.
constexpr int kLongThreads = 512;
constexpr int kLdsSlabs = 9;
template <typename T, int NREG, bool NT>
__global__ __launch_bounds__(kLongThreads) void ttt_loss_bwd_long_kernel(T* __restrict__ logits, const T* __restrict__ target,
                                                                         const float* __restrict__ grad, int vocab,
                                                                         int64_t z_stride, int64_t p_stride) {
    using LV = LossVec<T>;
    using raw = typename LV::raw;
    constexpr int N = LV::N;
    constexpr int SLAB = kLongThreads * N;
    constexpr int UNR = 4;
    extern __shared__ __align__(16) char smem[];
    __shared__ float red[3][kLongThreads / 64];
    const int tid = threadIdx.x;
    const int64_t row = blockIdx.x;
    T* z = logits + row * z_stride;
    const T* p = target + row * p_stride;
    const float g = grad[row];
    const int n_head = columns_before_boundary(z, vocab);
    z += n_head;
    p += n_head;
    vocab -= n_head;
    const int n_full = vocab / SLAB;                                              // >= 15
    const int n_lds = n_full > NREG ? min(n_full - NREG, kLdsSlabs) : 0;
    const int first_twice = NREG + n_lds;                                         // slabs from here on are read twice
    auto col = [&](int it) { return it * SLAB + tid * N; };
    raw* lds_z = reinterpret_cast<raw*>(smem) + tid;
    raw* lds_p = lds_z + kLdsSlabs * kLongThreads;

    LossSums<T> sums;
    for (int it = first_twice; it < n_full; it += UNR) {
        raw za[UNR], pa[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {   // past the last slab: that one again, not used
            za[u] = load_vec<T, false>(z, col(min(it + u, n_full - 1)));
            pa[u] = load_vec<T, false>(p, col(min(it + u, n_full - 1)));
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            if (it + u < n_full) sums.take(za[u], pa[u]);
    }
    for (int i = 0; i < n_lds; i += 3) {
        raw za[3], pa[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            za[u] = load_vec<T, NT>(z, col(NREG + min(i + u, n_lds - 1)));
            pa[u] = load_vec<T, NT>(p, col(NREG + min(i + u, n_lds - 1)));
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)
            if (i + u < n_lds) {
                lds_z[(i + u) * kLongThreads] = za[u];
                lds_p[(i + u) * kLongThreads] = pa[u];
                sums.take(za[u], pa[u]);
            }
    }
    raw zc[NREG], pc[NREG];
    const raw zt = load_edge<T, NT>(z, col(n_full), vocab, -INFINITY), pt = load_edge<T, NT>(p, col(n_full), vocab, 0.f);
#pragma unroll
    for (int it = 0; it < NREG; ++it) {
        zc[it] = load_vec<T, NT>(z, col(min(it, n_full - 1)));
        pc[it] = load_vec<T, NT>(p, col(min(it, n_full - 1)));
    }
    sums.take(zt, pt);
#pragma unroll
    for (int it = 0; it < NREG; ++it)
        if (it < n_full) sums.take(zc[it], pc[it]);
    if (tid < n_head) sums.take_one((float)z[tid - n_head], (float)p[tid - n_head]);

    float mc, w;
    sums.template finish<kLongThreads / 64>(red, g, mc, w);

    if (tid < n_head)
        z[tid - n_head] = (T)fmaf(fast_exp2(fmaf((float)z[tid - n_head], kLog2eL, -mc)), w, -(float)p[tid - n_head] * g);
    store_edge<T, NT>(z, col(n_full), vocab, loss_grad<T>(zt, pt, mc, w, g));
#pragma unroll
    for (int it = 0; it < NREG; ++it)
        if (it < n_full) store_vec<T, NT>(z, col(it), loss_grad<T>(zc[it], pc[it], mc, w, g));
    for (int i = 0; i < n_lds; ++i)
        store_vec<T, NT>(z, col(NREG + i), loss_grad<T>(lds_z[i * kLongThreads], lds_p[i * kLongThreads], mc, w, g));
    for (int it = first_twice; it < n_full; it += UNR) {
        raw za[UNR], pa[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            if (it + u < n_full) {
                za[u] = load_vec<T, NT>(z, col(it + u));
                pa[u] = load_vec<T, NT>(p, col(it + u));
            }
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            if (it + u < n_full) store_vec<T, NT>(z, col(it + u), loss_grad<T>(za[u], pa[u], mc, w, g));
    }
}

template <typename T, bool NT>
static hipError_t launch_loss_nt(T* z, const T* p, const float* grad, int64_t n_rows, int vocab, int64_t zs, int64_t ps,
                                 hipStream_t stream) {
    constexpr int N = LossVec<T>::N;
    const dim3 grid((unsigned)n_rows);
    ProfileScope prof("ttt_loss_bwd_kernel", stream);
    if (vocab <= kCacheIters * 256 * N) {
        hipLaunchKernelGGL((ttt_loss_bwd_kernel<T, 256, NT>), grid, dim3(256), 0, stream, z, p, grad, vocab, zs, ps);
    } else if (vocab <= kCacheIters * 512 * N) {
        hipLaunchKernelGGL((ttt_loss_bwd_kernel<T, 512, NT>), grid, dim3(512), 0, stream, z, p, grad, vocab, zs, ps);
    } else if (vocab <= kCacheIters * 1024 * N) {
        hipLaunchKernelGGL((ttt_loss_bwd_kernel<T, 1024, NT>), grid, dim3(1024), 0, stream, z, p, grad, vocab, zs, ps);
    } else {
        constexpr int LDS = 2 * kLdsSlabs * kLongThreads * 16;
        auto go = [&](auto kern, LdsOptIn& lds_opt_in) {
            if (hipError_t e = lds_opt_in.ensure((const void*)kern, LDS); e != hipSuccess) return e;
            hipLaunchKernelGGL(kern, grid, dim3(kLongThreads), LDS, stream, z, p, grad, vocab, zs, ps);
            return hipSuccess;
        };
        static LdsOptIn opt_in_18, opt_in_26;
        // 18 slabs in registers where all whole ones then fit
        const hipError_t e = vocab < (18 + kLdsSlabs + 1) * kLongThreads * N ? go(ttt_loss_bwd_long_kernel<T, 18, NT>, opt_in_18)
                                                                            : go(ttt_loss_bwd_long_kernel<T, 26, NT>, opt_in_26);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

// Logits and target together larger than the 256 MB memory-side cache: nothing of them is still there when it is
// used next, and accesses that pass the caches by are faster (28672 x 32000 fp32 2076 -> 1850 us, 8192 x 32000
// bf16 297 -> 270).  Below that they keep to the caches (8192 x 4096 fp32: 59 us, 65 passing by).
template <typename T>
static hipError_t launch_loss_t(void* logits, const void* target, const float* grad, int64_t n_rows, int vocab,
                                int64_t zs, int64_t ps, hipStream_t stream) {
    T* z = static_cast<T*>(logits);
    const T* p = static_cast<const T*>(target);
    if (2 * n_rows * vocab * (int64_t)sizeof(T) > (int64_t)256 << 20) return launch_loss_nt<T, true>(z, p, grad, n_rows, vocab, zs, ps, stream);
    return launch_loss_nt<T, false>(z, p, grad, n_rows, vocab, zs, ps, stream);
}

hipError_t launch_loss_bwd(int dtype, void* logits, const void* target, const float* grad, int64_t n_rows, int vocab,
                           int64_t zs, int64_t ps, hipStream_t stream) {
    if (dtype == TTT_BF16) return launch_loss_t<__bf16>(logits, target, grad, n_rows, vocab, zs, ps, stream);
    return launch_loss_t<float>(logits, target, grad, n_rows, vocab, zs, ps, stream);
}

}  // namespace ttt
