// The noise-free Grover search by the diffusion identity: a labelled variant of
// the HALL-based iteration, not the paper's form.
//
// One iteration is G = HALL . Inv . HALL . Oracle (Sec. 5.1).  With Inv =
// 2|0><0| - I (Eq. inversion) and HALL|0..0> = |s>, the uniform state (Eq.
// Shor1), HALL . Inv . HALL = 2|s><s| - I, so
//     (G C)_n = 2 m - (O C)_n,   m = mean over n of (O C)_n,
// where O flips the marked amplitudes.  Every unmarked amplitude thus changes sign
// and takes the same addend, every marked one takes the same addend without the
// sign: after k iterations
//     C_n -> (-1)^k C_n + a   (n not marked),     C_x -> C_x + b   (x marked).
// The two addends follow from the sums U over the unmarked and V over the marked
// amplitudes.  With |M| marked of N, the pair (U / sqrt(N - |M|), V / sqrt|M|) is
// rotated by one iteration through the angle t = 2 asin(sqrt(|M| / N)):
//     cos t = 1 - 2 |M| / N,   sin t = 2 sqrt(|M| (N - |M|)) / N
// (substitute m = (U - V) / N into U' = 2 m (N - |M|) - U and V' = V + 2 m |M|), so
// U and V after k iterations are the pair rotated by k t, and
//     a = (U_k - (-1)^k U) / (N - |M|),   b = (V_k - V) / |M|.
// The factors of U and V in them are computed on the host in twice double precision, by
// squaring the rotation: a sine of k t in double carries the rounding of t k times (N =
// 16, k = 3000: error 7.0e-14, iteration by iteration 5.8e-15, now 3e-16).
// The state is read once for U and read and written once for the result, whatever
// k is; all of it in FP64 (also for FP32 states), sums in a fixed order.  Iteration by
// iteration (one pass and one combining launch each), the n_q = 20 search took 8.46
// ms; this takes 21 us, three launches' latency.
#include <hip/hip_runtime.h>

#include <cmath>

#include "pk_launch.h"

namespace pk {

namespace {

constexpr int kThreads = 256;
constexpr int kGrid = 2048;  // blocks of the streaming kernels (and partial sums)

template <typename T>
__device__ __forceinline__ double2 wide(const T& v) {
    return double2{(double)v.x, (double)v.y};
}

// Sum of a block's values (FP64), written to part[blockIdx.x] by thread 0.
__device__ __forceinline__ void block_sum2(double2 acc, double2* part) {
    __shared__ double2 red[kThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        acc.x += __shfl_xor(acc.x, off, 64);
        acc.y += __shfl_xor(acc.y, off, 64);
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double2 t = {0.0, 0.0};
        for (int w = 0; w < kThreads / 64; ++w) {
            t.x += red[w].x;
            t.y += red[w].y;
        }
        part[blockIdx.x] = t;
    }
}

// Block b owns the contiguous chunk [b * chunk, (b + 1) * chunk) of the state.
template <typename T>
__global__ void __launch_bounds__(kThreads) sum_kernel(const T* src, int64_t n, int64_t chunk, double2* part) {
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    double2 acc = {0.0, 0.0};
#pragma unroll 4
    for (int64_t e = lo + threadIdx.x; e < hi; e += kThreads) {
        const double2 v = wide(src[e]);
        acc.x += v.x;
        acc.y += v.y;
    }
    block_sum2(acc, part);
}

// The addends of k iterations from the sums: a = uu U - w V, b = vv V + w U.
struct Rotation {
    double uu, w, vv;
    int many;  // k > 1
};

struct Addends {
    double2 a, b;
};

__device__ __forceinline__ Addends addends(double2 sum, double2 V, const Rotation& q) {
    const double2 U = {sum.x - V.x, sum.y - V.y};
    Addends r;
    r.a = double2{q.uu * U.x, q.uu * U.y};
    r.b = double2{q.vv * V.x, q.vv * V.y};
    if (q.w != 0.0) {  // else none or all are marked, and U or V is no sum of amplitudes
        r.a.x -= q.w * V.x;
        r.a.y -= q.w * V.y;
        r.b.x += q.w * U.x;
        r.b.y += q.w * U.y;
    }
    // from the second iteration on, the mean of a non-finite part is NaN
    if (q.many && !isfinite(sum.x)) r.a.x = r.b.x = __builtin_nan("");
    if (q.many && !isfinite(sum.y)) r.a.y = r.b.y = __builtin_nan("");
    return r;
}

template <typename T>
__device__ __forceinline__ T plus(const T& v, double sign, const double2& add) {
    using R = decltype(v.x);
    T w;
    w.x = (R)(sign * (double)v.x + add.x);
    w.y = (R)(sign * (double)v.y + add.y);
    return w;
}

// One workgroup: the block sums added in order (lane l adds parts l, l + 64, ..., then
// a butterfly), the addends, and L = sum_x |C_x + b|^2 of the values that
// apply_kernel will store.
template <typename T>
__global__ void __launch_bounds__(64) combine_kernel(const double2* part, int nparts, MarkedSet ms, const T* src,
                                                     Rotation q, double2* add, double* L) {
    // all of a lane's loads are issued before the first add, so their latencies overlap
    constexpr int kPer = kGrid / 64;
    const int lane = threadIdx.x;
    T own{0, 0};
    if (lane < ms.count) own = src[ms.label[lane]];
    double2 pv[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int b = lane + 64 * j;
        pv[j] = b < nparts ? part[b] : double2{0.0, 0.0};
    }
    double2 s = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (lane + 64 * j < nparts) {
            s.x += pv[j].x;
            s.y += pv[j].y;
        }
    double2 v = wide(own);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s.x += __shfl_xor(s.x, off, 64);
        s.y += __shfl_xor(s.y, off, 64);
        v.x += __shfl_xor(v.x, off, 64);
        v.y += __shfl_xor(v.y, off, 64);
    }
    const Addends r = addends(s, v, q);
    const double2 c = wide(plus(own, 1.0, r.b));
    double l = lane < ms.count ? c.x * c.x + c.y * c.y : 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0) {
        add[0] = r.a;
        add[1] = r.b;
        *L = l;
    }
}

// The result, chunk by chunk; only a chunk that holds marked labels looks for them.
template <typename T>
__global__ void __launch_bounds__(kThreads) apply_kernel(const T* src, T* dst, int64_t n, int64_t chunk, double sign,
                                                         const double2* add, MarkedSet ms) {
    const double2 a = add[0], b = add[1];
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    bool any = false;
    for (int i = 0; i < ms.count; ++i) any = any || (ms.label[i] >= lo && ms.label[i] < hi);
    if (!any) {
#pragma unroll 4
        for (int64_t e = lo + threadIdx.x; e < hi; e += kThreads) dst[e] = plus(src[e], sign, a);
    } else {
        for (int64_t e = lo + threadIdx.x; e < hi; e += kThreads) {
            bool marked = false;
            for (int i = 0; i < ms.count; ++i) marked = marked || e == ms.label[i];
            dst[e] = marked ? plus(src[e], 1.0, b) : plus(src[e], sign, a);
        }
    }
}

// States that one workgroup holds in registers (up to kSmall amplitudes): the sum, the
// addends and the result in one launch.
constexpr int64_t kSmall = 16 * kThreads;

template <typename T>
__global__ void __launch_bounds__(kThreads) small_kernel(const T* src, T* dst, int64_t n, double sign, Rotation q,
                                                         MarkedSet ms, double* L) {
    constexpr int kPer = (int)(kSmall / kThreads), nw = kThreads / 64;
    __shared__ double2 red[2][nw];
    __shared__ double lred[nw];
    T v[kPer];
    unsigned marked = 0;
    double2 s = {0.0, 0.0}, m = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t e = threadIdx.x + kThreads * j;
        v[j] = T{0, 0};
        if (e >= n) continue;
        v[j] = src[e];
        for (int i = 0; i < ms.count; ++i)
            if (e == ms.label[i]) marked |= 1u << j;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const double2 w = wide(v[j]);
        s.x += w.x;
        s.y += w.y;
        if (marked >> j & 1u) {
            m.x += w.x;
            m.y += w.y;
        }
    }
    auto total = [&](double2 x, double2* r) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            x.x += __shfl_xor(x.x, off, 64);
            x.y += __shfl_xor(x.y, off, 64);
        }
        if ((threadIdx.x & 63) == 0) r[threadIdx.x >> 6] = x;
        __syncthreads();
        double2 t = {0.0, 0.0};
#pragma unroll
        for (int w = 0; w < nw; ++w) {
            t.x += r[w].x;
            t.y += r[w].y;
        }
        return t;
    };
    const double2 sum = total(s, red[0]), V = total(m, red[1]);
    const Addends r = addends(sum, V, q);
    double l = 0.0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t e = threadIdx.x + kThreads * j;
        if (e >= n) continue;
        const bool hit = marked >> j & 1u;
        const T w = hit ? plus(v[j], 1.0, r.b) : plus(v[j], sign, r.a);
        dst[e] = w;
        const double2 c = wide(w);
        if (hit) l += c.x * c.x + c.y * c.y;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if ((threadIdx.x & 63) == 0) lred[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < nw; ++w) t += lred[w];
        *L = t;
    }
}

// A number as the sum of two doubles, the second below half an ulp of the first.
struct Twice {
    double hi, lo;
};

Twice sum2(double a, double b) {
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}

Twice operator+(Twice a, Twice b) {
    const Twice s = sum2(a.hi, b.hi);
    return sum2(s.hi, s.lo + a.lo + b.lo);
}

Twice operator-(Twice a) { return {-a.hi, -a.lo}; }

Twice operator*(Twice a, Twice b) {
    const double p = a.hi * b.hi;
    return sum2(p, std::fma(a.hi, b.hi, -p) + a.hi * b.lo + a.lo * b.hi);
}

// The k-th power of the rotation of one iteration, whose cosine is exact in double, as
// the factors of Rotation.  Its angle's error grows as k 2^-104.
Rotation rotation(int64_t n, int count, int64_t k) {
    const double N = (double)n, M = (double)count, K = N - M, odd = (k & 1) ? 1.0 : 0.0;
    const int many = k > 1;
    if (count == 0) return {2.0 * odd / N, 0.0, 0.0, many};   // the mean does not change
    if (count == n) return {0.0, 0.0, -2.0 * odd / N, many};  // m = -V / N, the sign of V alternates
    const double root = std::sqrt(M * K);  // M K is exact: below 2^37
    const Twice g = sum2(root, std::fma(-root, root, M * K) / (2.0 * root));
    Twice c = {1.0 - 2.0 * M / N, 0.0}, s = {2.0 * g.hi / N, 2.0 * g.lo / N};
    Twice ck = {1.0, 0.0}, sk = {0.0, 0.0};
    for (int64_t e = k; e; e >>= 1) {
        if (e & 1) {
            const Twice t = ck * c + -(sk * s);
            sk = sk * c + ck * s;
            ck = t;
        }
        const Twice t = c * c + -(s * s);
        s = c * s;
        s = {2.0 * s.hi, 2.0 * s.lo};
        c = t;
    }
    const Twice up = ck + Twice{odd > 0.0 ? 1.0 : -1.0, 0.0}, down = ck + Twice{-1.0, 0.0};
    return {(up.hi + up.lo) / K, (sk.hi + sk.lo) / root, (down.hi + down.lo) / M, many};
}

template <typename T>
hipError_t search_t(const void* psi_in, void* psi_out, int64_t n, const MarkedSet& ms, int64_t iters,
                    double2* part, double2* add, double* L, hipStream_t st) {
    const T* in = static_cast<const T*>(psi_in);
    T* out = static_cast<T*>(psi_out);
    const Rotation q = rotation(n, ms.count, iters);
    const double sign = (iters & 1) ? -1.0 : 1.0;
    if (n <= kSmall) {
        hipLaunchKernelGGL(small_kernel<T>, dim3(1), dim3(kThreads), 0, st, in, out, n, sign, q, ms, L);
        return hipGetLastError();
    }
    // at least four amplitudes a thread, at most kGrid blocks
    int64_t chunk = (n + kGrid - 1) / kGrid;
    if (chunk < 4 * kThreads) chunk = 4 * kThreads;
    const int grid = (int)((n + chunk - 1) / chunk);
    hipLaunchKernelGGL(sum_kernel<T>, dim3(grid), dim3(kThreads), 0, st, in, n, chunk, part);
    hipLaunchKernelGGL(combine_kernel<T>, dim3(1), dim3(64), 0, st, part, grid, ms, in, q, add, L);
    hipLaunchKernelGGL(apply_kernel<T>, dim3(grid), dim3(kThreads), 0, st, in, out, n, chunk, sign, add,
                       ms);
    return hipGetLastError();
}

}  // namespace

size_t search_workspace_bytes() { return (size_t)(kGrid + 2) * sizeof(double2); }

hipError_t launch_search(const void* psi_in, void* psi_out, int nq, bool fp64, const MarkedSet& ms, int64_t iters,
                         void* workspace, double* L, hipStream_t st) {
    double2* part = static_cast<double2*>(workspace);
    double2* add = part + kGrid;
    const int64_t n = (int64_t)1 << nq;
    return fp64 ? search_t<double2>(psi_in, psi_out, n, ms, iters, part, add, L, st)
                : search_t<float2>(psi_in, psi_out, n, ms, iters, part, add, L, st);
}

}  // namespace pk
