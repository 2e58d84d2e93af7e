// BLAS-1 kernels and the device-resident Krylov scalar algebra.
//
// Reductions are deterministic and fence-free: the partial kernel reduces each
// block with wavefront shuffles (64 lanes) and a fixed-order sum over its four
// waves and writes one partial per quantity; a one-block-per-column finaliser
// (the next launch, so the kernel boundary orders the two) adds the partials
// in block order and turns the sums into Krylov coefficients.  No cross-block
// fence is needed inside a kernel, which matters on a part whose L2 caches are
// private to each XCD.  The host never has to read a scalar back to continue:
// CG, CGNR and GCR coefficients live on the device and a per-column `done` /
// `stop` flag turns later updates into no-ops.  Accumulation is FP64 for both
// FP32 and FP64 vectors.
#include <utility>

#include <algorithm>

#include "kernels.hpp"

namespace dwf {

namespace {

constexpr int kWaves = kBlock / 64;
constexpr int kMaxQ = 40;

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    return x;
}

// Reduce per-thread values v[0..nq) over the block; totals end in tot[0..nq)
// (shared) and are visible to every thread of the block afterwards.
template <int NQ>
__device__ __forceinline__ void block_reduce(double (&v)[NQ], int nq, double* sh, double* tot) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q < nq) {
            double s = wave_sum(v[q]);
            if (lane == 0) sh[q * kWaves + wid] = s;
        }
    }
    __syncthreads();
    if (threadIdx.x < nq) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s += sh[threadIdx.x * kWaves + w];
        tot[threadIdx.x] = s;
    }
    __syncthreads();
}

template <int NQ>
__device__ __forceinline__ void write_partials(double (&v)[NQ], int nq, const RedWork& rw, int col, double* sh,
                                               double* tot) {
    block_reduce<NQ>(v, nq, sh, tot);
    double* part = rw.partial + (size_t)col * rw.max_q * rw.nblk;
    if (threadIdx.x < nq) part[(size_t)threadIdx.x * rw.nblk + blockIdx.x] = tot[threadIdx.x];
}

// finaliser side: column `col` (= blockIdx.x), nb partials per quantity
template <int NQ>
__device__ __forceinline__ void sum_partials(int nq, int nb, const RedWork& rw, int col, double* sh, double* tot) {
    const double* part = rw.partial + (size_t)col * rw.max_q * rw.nblk;
    double w[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        w[q] = 0.0;
        if (q < nq)
            for (int b = threadIdx.x; b < nb; b += blockDim.x) w[q] += part[(size_t)q * rw.nblk + b];
    }
    block_reduce<NQ>(w, nq, sh, tot);
}

// at least two entries per thread: a block's partial sums cost about as much as
// streaming a few thousand entries, so small vectors take fewer, fuller blocks
inline dim3 red_grid(size_t n, int ncol, const RedWork& rw) {
    long long nb = (long long)((n + 2 * kBlock - 1) / (2 * kBlock));
    if (nb > rw.nblk) nb = rw.nblk;
    if (nb < 1) nb = 1;
    return dim3((unsigned)nb, (unsigned)ncol);
}

inline dim3 ew_grid(size_t n, int ncol) {
    long long nb = (long long)((n + kBlock - 1) / kBlock);
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    return dim3((unsigned)nb, (unsigned)ncol);
}

#define GRID_STRIDE(i, n) \
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (size_t)gridDim.x * blockDim.x)

#define SHARED_RED __shared__ double sh[kMaxQ * kWaves], tot[kMaxQ]

// calls f(std::integral_constant<int, j>) for a run-time j in Js...
template <typename F, int... Js>
void with_j(int j, F&& f, std::integer_sequence<int, Js...>) {
    ((j == Js ? (f(std::integral_constant<int, Js>{}), 0) : 0), ...);
}


template <typename T>
__device__ __forceinline__ cpx<double> up(cpx<T> a) { return {(double)a.re, (double)a.im}; }

__device__ __forceinline__ bool finite(double x) { return !(isnan(x) || isinf(x)); }

}  // namespace

// ------------------------------------------------------------ elementwise
template <typename T>
__global__ void k_zero(cpx<T>* x, size_t n) {
    GRID_STRIDE(i, n) x[i] = {T(0), T(0)};
}
template <typename Ti, typename To>
__global__ void k_convert(const cpx<Ti>* in, cpx<To>* out, size_t n) {
    GRID_STRIDE(i, n) out[i] = {(To)in[i].re, (To)in[i].im};
}
template <typename Tx, typename Ty>
__global__ void k_add(const cpx<Tx>* x, cpx<Ty>* y, size_t n) {
    GRID_STRIDE(i, n) {
        cpx<Ty> a = y[i];
        y[i] = {a.re + (Ty)x[i].re, a.im + (Ty)x[i].im};
    }
}
template <typename T>
__global__ void k_sub(const cpx<T>* a, const cpx<T>* b, cpx<T>* out, size_t n) {
    GRID_STRIDE(i, n) out[i] = a[i] - b[i];
}

// y = a x + b y (b == 0: y = a x, whatever y held)
template <typename T>
__global__ void k_axpby(double a, const cpx<T>* x, double b, cpx<T>* y, size_t n) {
    const T ta = (T)a, tb = (T)b;
    if (b == 0.0) {
        GRID_STRIDE(i, n) y[i] = ta * x[i];
    } else {
        GRID_STRIDE(i, n) y[i] = ta * x[i] + tb * y[i];
    }
}
template <typename T> hipError_t vaxpby(double a, const cpx<T>* x, double b, cpx<T>* y, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_axpby<T>, ew_grid(n, 1), dim3(kBlock), 0, st, a, x, b, y, n);
    return hipGetLastError();
}
template hipError_t vaxpby<float>(double, const cpx<float>*, double, cpx<float>*, size_t, hipStream_t);
template hipError_t vaxpby<double>(double, const cpx<double>*, double, cpx<double>*, size_t, hipStream_t);

template <typename T> hipError_t vzero(cpx<T>* x, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_zero<T>, ew_grid(n, 1), dim3(kBlock), 0, st, x, n);
    return hipGetLastError();
}
template <typename Ti, typename To>
hipError_t vconvert(const cpx<Ti>* in, cpx<To>* out, size_t n, hipStream_t st) {
    hipLaunchKernelGGL((k_convert<Ti, To>), ew_grid(n, 1), dim3(kBlock), 0, st, in, out, n);
    return hipGetLastError();
}
template <typename Tx, typename Ty>
hipError_t vadd(const cpx<Tx>* x, cpx<Ty>* y, size_t n, hipStream_t st) {
    hipLaunchKernelGGL((k_add<Tx, Ty>), ew_grid(n, 1), dim3(kBlock), 0, st, x, y, n);
    return hipGetLastError();
}
template <typename T>
hipError_t vsub(const cpx<T>* a, const cpx<T>* b, cpx<T>* out, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_sub<T>, ew_grid(n, 1), dim3(kBlock), 0, st, a, b, out, n);
    return hipGetLastError();
}

// ------------------------------------------------------------ streaming copy (bandwidth reference)
// dst = src in 16-byte words: each workgroup copies one contiguous chunk of
// 1024 words (16 KB), every thread issuing its four loads before its four
// nontemporal stores.  Of the copy forms measured on the MI355X (grid-stride
// loops with 1 k - 8 k workgroups, chunks of 1 k - 16 k words with 4 - 16 loads
// in flight, with and without nontemporal loads and stores, hipMemcpyAsync),
// this one moved the most bytes per second over 2 GiB.
typedef unsigned int sc_u32x4 __attribute__((ext_vector_type(4)));
constexpr int kCopyChunk = 1024;
__global__ void __launch_bounds__(kBlock) k_stream_copy(const sc_u32x4* __restrict__ src, sc_u32x4* __restrict__ dst,
                                                        size_t n) {
    const size_t base = (size_t)blockIdx.x * kCopyChunk;
    if (base + kCopyChunk <= n) {
        sc_u32x4 v[kCopyChunk / kBlock];
#pragma unroll
        for (int u = 0; u < kCopyChunk / kBlock; ++u) v[u] = src[base + u * kBlock + threadIdx.x];
#pragma unroll
        for (int u = 0; u < kCopyChunk / kBlock; ++u)
            __builtin_nontemporal_store(v[u], dst + base + u * kBlock + threadIdx.x);
    } else {
        for (size_t i = base + threadIdx.x; i < n; i += kBlock) dst[i] = src[i];
    }
}

hipError_t stream_copy(const void* src, void* dst, size_t words, hipStream_t st) {
    const size_t blocks = (words + kCopyChunk - 1) / kCopyChunk;
    if (blocks == 0 || blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_stream_copy, dim3((unsigned)blocks), dim3(kBlock), 0, st,
                       reinterpret_cast<const sc_u32x4*>(src), reinterpret_cast<sc_u32x4*>(dst), words);
    return hipGetLastError();
}

// ------------------------------------------------------------ finalisers (one block per column)
// out[col * stride + q] = total q
__global__ void __launch_bounds__(kBlock) k_fin_store(RedWork rw, int nq, int nb, double* out, size_t stride) {
    SHARED_RED;
    const int col = blockIdx.x;
    sum_partials<kMaxQ>(nq, nb, rw, col, sh, tot);
    if (threadIdx.x < nq) out[(size_t)col * stride + threadIdx.x] = tot[threadIdx.x];
}

// the same sums with one block per (quantity, column): for many quantities
// the same with one wavefront per (quantity, column): no barrier, all loads in flight
__global__ void __launch_bounds__(64) k_fin_store_q1(RedWork rw, int nb, double* out, size_t stride) {
    const int q = blockIdx.x, col = blockIdx.y;
    const double* part = rw.partial + (size_t)col * rw.max_q * rw.nblk + (size_t)q * rw.nblk;
    double s = 0.0;
#pragma unroll 8
    for (int b = threadIdx.x; b < nb; b += 64) s += part[b];
    s = wave_sum(s);
    if (threadIdx.x == 0) out[(size_t)col * stride + q] = s;
}

__global__ void __launch_bounds__(kBlock) k_fin_store_q(RedWork rw, int nb, double* out, size_t stride) {
    __shared__ double sh[kWaves];
    const int q = blockIdx.x, col = blockIdx.y;
    const double* part = rw.partial + (size_t)col * rw.max_q * rw.nblk + (size_t)q * rw.nblk;
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) s += part[b];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += sh[w];
        out[(size_t)col * stride + q] = t;
    }
}

__global__ void __launch_bounds__(kBlock) k_fin_cg_init(RedWork rw, int nb, CgScal* s, double tol2) {
    SHARED_RED;
    const int col = blockIdx.x;
    sum_partials<1>(1, nb, rw, col, sh, tot);
    if (threadIdx.x == 0) {
        CgScal c;
        c.zz = tot[0];
        c.zz0 = tot[0];
        c.alpha = 0.0;
        c.beta = 0.0;
        c.tol2 = tol2;
        c.iters = 0;
        c.done = (tot[0] == 0.0) ? 1 : (finite(tot[0]) ? 0 : 4);
        s[col] = c;
    }
}

__global__ void __launch_bounds__(kBlock) k_fin_cg_alpha(RedWork rw, int nb, CgScal* s) {
    SHARED_RED;
    const int col = blockIdx.x;
    if (s[col].done) return;
    sum_partials<1>(1, nb, rw, col, sh, tot);
    if (threadIdx.x == 0) {
        const double ww = tot[0];
        if (!(ww > 0.0) || !finite(ww)) {
            s[col].alpha = 0.0;
            s[col].done = finite(ww) ? 2 : 4;   // breakdown / non-finite
        } else {
            s[col].alpha = s[col].zz / ww;
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_fin_cg_beta(RedWork rw, int nb, CgScal* s, int maxit) {
    SHARED_RED;
    const int col = blockIdx.x;
    if (s[col].done) return;
    sum_partials<1>(1, nb, rw, col, sh, tot);
    if (threadIdx.x == 0) {
        CgScal c = s[col];
        const double znew = tot[0];
        c.iters += 1;
        if (!finite(znew)) {
            c.done = 4;
        } else {
            c.beta = znew / c.zz;
            c.zz = znew;
            if (znew <= c.tol2 * c.zz0) c.done = 1;
            else if (c.iters >= maxit) c.done = 3;
        }
        s[col] = c;
    }
}

// ------------------------------------------------------------ reductions: partial kernels
template <typename T>
__global__ void __launch_bounds__(kBlock) k_norm2_part(const cpx<T>* x, size_t n, RedWork rw, const int* skip, int sks) {
    SHARED_RED;
    const int col = blockIdx.y;
    if (skip && skip[(size_t)col * sks]) return;
    const cpx<T>* xc = x + (size_t)col * n;
    double v[1] = {0.0};
    GRID_STRIDE(i, n) {
        cpx<double> a = up(xc[i]);
        v[0] += a.re * a.re + a.im * a.im;
    }
    write_partials<1>(v, 1, rw, col, sh, tot);
}

template <typename T>
__global__ void __launch_bounds__(kBlock) k_cdot_part(const cpx<T>* a, const cpx<T>* b, size_t n, RedWork rw) {
    SHARED_RED;
    const int col = blockIdx.y;
    const cpx<T>* ac = a + (size_t)col * n;
    const cpx<T>* bc = b + (size_t)col * n;
    double v[2] = {0.0, 0.0};
    GRID_STRIDE(i, n) {
        cpx<double> p = cjmul(up(ac[i]), up(bc[i]));
        v[0] += p.re;
        v[1] += p.im;
    }
    write_partials<2>(v, 2, rw, col, sh, tot);
}

namespace {
const int kCgSkipStride = (int)(sizeof(CgScal) / sizeof(int));
}

template <typename T>
hipError_t norm2(const cpx<T>* x, size_t n, int ncol, double* out, const RedWork& rw, hipStream_t st) {
    dim3 g = red_grid(n, ncol, rw);
    hipLaunchKernelGGL(k_norm2_part<T>, g, dim3(kBlock), 0, st, x, n, rw, (const int*)nullptr, 1);
    hipLaunchKernelGGL(k_fin_store, dim3(ncol), dim3(kBlock), 0, st, rw, 1, (int)g.x, out, (size_t)1);
    return hipGetLastError();
}
template <typename T>
hipError_t cdot(const cpx<T>* a, const cpx<T>* b, size_t n, int ncol, double* out2, const RedWork& rw, hipStream_t st) {
    dim3 g = red_grid(n, ncol, rw);
    hipLaunchKernelGGL(k_cdot_part<T>, g, dim3(kBlock), 0, st, a, b, n, rw);
    hipLaunchKernelGGL(k_fin_store, dim3(ncol), dim3(kBlock), 0, st, rw, 2, (int)g.x, out2, (size_t)2);
    return hipGetLastError();
}

// ------------------------------------------------------------ CG family
template <typename T>
hipError_t cg_init(const cpx<T>* v, size_t n, int ncol, CgScal* s, double tol, const RedWork& rw, hipStream_t st) {
    dim3 g = red_grid(n, ncol, rw);
    hipLaunchKernelGGL(k_norm2_part<T>, g, dim3(kBlock), 0, st, v, n, rw, (const int*)nullptr, 1);
    hipLaunchKernelGGL(k_fin_cg_init, dim3(ncol), dim3(kBlock), 0, st, rw, (int)g.x, s, tol * tol);
    return hipGetLastError();
}
template <typename T>
hipError_t cg_alpha(const cpx<T>* w, size_t n, int ncol, CgScal* s, const RedWork& rw, hipStream_t st) {
    dim3 g = red_grid(n, ncol, rw);
    hipLaunchKernelGGL(k_norm2_part<T>, g, dim3(kBlock), 0, st, w, n, rw, &s[0].done, kCgSkipStride);
    hipLaunchKernelGGL(k_fin_cg_alpha, dim3(ncol), dim3(kBlock), 0, st, rw, (int)g.x, s);
    return hipGetLastError();
}

template <typename T>
__global__ void k_cg_update_xr(cpx<T>* x, cpx<T>* r, const cpx<T>* p, const cpx<T>* w, size_t n, const CgScal* s) {
    const int col = blockIdx.y;
    if (s[col].done) return;
    const T a = (T)s[col].alpha;
    const size_t o = (size_t)col * n;
    GRID_STRIDE(i, n) {
        cpx<T> pi = p[o + i], wi = w[o + i], xi = x[o + i], ri = r[o + i];
        x[o + i] = {xi.re + a * pi.re, xi.im + a * pi.im};
        r[o + i] = {ri.re - a * wi.re, ri.im - a * wi.im};
    }
}

template <typename T>
__global__ void k_cg_update_p(cpx<T>* p, const cpx<T>* z, size_t n, const CgScal* s) {
    const int col = blockIdx.y;
    if (s[col].done) return;
    const T b = (T)s[col].beta;
    const size_t o = (size_t)col * n;
    GRID_STRIDE(i, n) {
        cpx<T> pi = p[o + i], zi = z[o + i];
        p[o + i] = {zi.re + b * pi.re, zi.im + b * pi.im};
    }
}

template <typename T>
hipError_t cg_update_xr(cpx<T>* x, cpx<T>* r, const cpx<T>* p, const cpx<T>* w, size_t n, int ncol,
                        const CgScal* s, hipStream_t st) {
    hipLaunchKernelGGL(k_cg_update_xr<T>, ew_grid(n, ncol), dim3(kBlock), 0, st, x, r, p, w, n, s);
    return hipGetLastError();
}
template <typename T>
hipError_t cg_beta(const cpx<T>* z, size_t n, int ncol, CgScal* s, int maxit, const RedWork& rw, hipStream_t st) {
    dim3 g = red_grid(n, ncol, rw);
    hipLaunchKernelGGL(k_norm2_part<T>, g, dim3(kBlock), 0, st, z, n, rw, &s[0].done, kCgSkipStride);
    hipLaunchKernelGGL(k_fin_cg_beta, dim3(ncol), dim3(kBlock), 0, st, rw, (int)g.x, s, maxit);
    return hipGetLastError();
}
template <typename T>
hipError_t cg_update_p(cpx<T>* p, const cpx<T>* z, size_t n, int ncol, const CgScal* s, hipStream_t st) {
    hipLaunchKernelGGL(k_cg_update_p<T>, ew_grid(n, ncol), dim3(kBlock), 0, st, p, z, n, s);
    return hipGetLastError();
}

// ------------------------------------------------------------ CGNR (coarsest level)
// A finaliser per inner product cost two of ten launches an iteration, 1.7 us each on a coarsest
// level of 256 sites where a whole iteration took 30 us; here every workgroup adds the partials
// (L2 hits, at most a few tens of KB) and the column's first workgroup passes the state on in a
// second buffer.  The norms' passes over the vectors are gone too: the stencils leave the partials.
// All first loads - partials, state, fields - are issued before any is waited for, the state field by
// field: with the state as a local struct (which the compiler put in LDS) and the partials
// loaded behind it, x and r took 7.8 us on 256 sites x 8 slices x 16; now 2.8, p 2.6.  An iteration
// there takes six launches, 22 us against 30 with ten.
namespace {
constexpr int kPartBatch = 8;   // partials per thread in flight
struct PartLoads {
    double v[kPartBatch];
};
__device__ __forceinline__ PartLoads partials_load(const double* part, int np) {
    PartLoads l;
#pragma unroll
    for (int j = 0; j < kPartBatch; ++j) {
        const int b = (int)threadIdx.x + j * kBlock;
        l.v[j] = part[b < np ? b : 0];
    }
    return l;
}
__device__ __forceinline__ double partials_total(const PartLoads& l, const double* part, int np, double* sh) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < kPartBatch; ++j) t += (int)threadIdx.x + j * kBlock < np ? l.v[j] : 0.0;
    for (int b = threadIdx.x + kPartBatch * kBlock; b < np; b += kBlock) t += part[b];
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = t;
    __syncthreads();
    t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += sh[w];
    return t;
}
}  // namespace

template <typename T>
__global__ void __launch_bounds__(kBlock)
k_cgnr_xr(cpx<T>* x, cpx<T>* r, const cpx<T>* p, const cpx<T>* q, size_t n, const CgScal* s, double* s2,
          const double* part, size_t pstride, int np) {
    __shared__ double sh[kWaves];
    const int col = blockIdx.y;
    const size_t o = (size_t)col * n, stride = (size_t)gridDim.x * kBlock;
    size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const size_t e0 = e < n ? e : 0;
    const double* pc = part + (size_t)col * pstride;
    const PartLoads pl = partials_load(pc, np);
    const CgScal* sc = s + col;
    const double zz = sc->zz, zz0 = sc->zz0, tol2 = sc->tol2, beta = sc->beta;
    const int iters = sc->iters;
    int done = sc->done;
    double alpha = sc->alpha;
    cpx<T> pi = p[o + e0], qi = q[o + e0], xi = x[o + e0], ri = r[o + e0];
    const double ww = partials_total(pl, pc, np, sh);
    if (done == 0) {
        alpha = zz / ww;
        if (!(ww > 0.0) || !finite(ww)) {
            alpha = 0.0;
            done = finite(ww) ? 2 : 4;   // breakdown / non-finite
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        CgScal* d = reinterpret_cast<CgScal*>(s2 + (size_t)col * pstride);
        d->zz = zz;
        d->zz0 = zz0;
        d->tol2 = tol2;
        d->alpha = alpha;
        d->beta = beta;
        d->done = done;
        d->iters = iters;
    }
    if (done) return;
    const T a = (T)alpha;
    while (e < n) {
        x[o + e] = {xi.re + a * pi.re, xi.im + a * pi.im};
        r[o + e] = {ri.re - a * qi.re, ri.im - a * qi.im};
        e += stride;
        if (e < n) { pi = p[o + e]; qi = q[o + e]; xi = x[o + e]; ri = r[o + e]; }
    }
}

template <typename T>
__global__ void __launch_bounds__(kBlock)
k_cgnr_p(cpx<T>* p, const cpx<T>* z, size_t n, int maxit, const double* s2, CgScal* s, const double* part, size_t pstride,
         int np) {
    __shared__ double sh[kWaves];
    const int col = blockIdx.y;
    const size_t o = (size_t)col * n, stride = (size_t)gridDim.x * kBlock;
    size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const size_t e0 = e < n ? e : 0;
    const double* pc = part + (size_t)col * pstride;
    const PartLoads pl = partials_load(pc, np);
    const CgScal* sc = reinterpret_cast<const CgScal*>(s2 + (size_t)col * pstride);
    const double zz0 = sc->zz0, tol2 = sc->tol2, alpha = sc->alpha;
    double zz = sc->zz, beta = sc->beta;
    int done = sc->done, iters = sc->iters;
    cpx<T> pi = p[o + e0], zi = z[o + e0];
    const double znew = partials_total(pl, pc, np, sh);
    if (done == 0) {
        iters += 1;
        if (!finite(znew)) {
            done = 4;
        } else {
            beta = znew / zz;
            zz = znew;
            if (znew <= tol2 * zz0) done = 1;
            else if (iters >= maxit) done = 3;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        CgScal* d = s + col;
        d->zz = zz;
        d->zz0 = zz0;
        d->tol2 = tol2;
        d->alpha = alpha;
        d->beta = beta;
        d->done = done;
        d->iters = iters;
    }
    if (done) return;
    const T b = (T)beta;
    while (e < n) {
        p[o + e] = {zi.re + b * pi.re, zi.im + b * pi.im};
        e += stride;
        if (e < n) { pi = p[o + e]; zi = z[o + e]; }
    }
}

namespace {
// workgroups of the updates: one entry per thread while the chip has room, then several (each
// workgroup adds the partials once)
inline dim3 cgnr_grid(size_t n, int ncol) {
    const size_t nb = (n + kBlock - 1) / kBlock;
    return dim3((unsigned)std::max<size_t>(1, std::min<size_t>(nb, std::max(1024 / ncol, 64))), (unsigned)ncol);
}
}  // namespace

template <typename T>
hipError_t cgnr_xr(cpx<T>* x, cpx<T>* r, const cpx<T>* p, const cpx<T>* q, size_t n, int ncol, const CgScal* s, double* s2,
                   const double* part, size_t pstride, int np, hipStream_t st) {
    hipLaunchKernelGGL(k_cgnr_xr<T>, cgnr_grid(n, ncol), dim3(kBlock), 0, st, x, r, p, q, n, s, s2, part, pstride, np);
    return hipGetLastError();
}
template <typename T>
hipError_t cgnr_p(cpx<T>* p, const cpx<T>* z, size_t n, int ncol, int maxit, const double* s2, CgScal* s, const double* part,
                  size_t pstride, int np, hipStream_t st) {
    hipLaunchKernelGGL(k_cgnr_p<T>, cgnr_grid(n, ncol), dim3(kBlock), 0, st, p, z, n, maxit, s2, s, part, pstride, np);
    return hipGetLastError();
}
template <typename T>
hipError_t norm2_partials(const cpx<T>* x, size_t n, int ncol, const CgScal* s, double* part, size_t pstride, int* np,
                          hipStream_t st) {
    // k_norm2_part with its partials at `part` (one quantity per column, pstride apart)
    RedWork rw;
    rw.partial = part;
    rw.nblk = (int)pstride;
    rw.max_q = 1;
    rw.max_cols = ncol;
    const unsigned nb = (unsigned)std::max<size_t>(1, std::min<size_t>((n + 2 * kBlock - 1) / (2 * kBlock), 512));
    *np = (int)nb;
    hipLaunchKernelGGL(k_norm2_part<T>, dim3(nb, ncol), dim3(kBlock), 0, st, x, n, rw, &s[0].done, kCgSkipStride);
    return hipGetLastError();
}

// ------------------------------------------------------------ GCR
namespace {
__device__ __forceinline__ cpx<double> ld2(const double* p) { return {p[0], p[1]}; }
// entries per thread whose loads the fused GCR kernels issue together (bounded by
// the registers of U (j + 2) loaded vectors)
template <typename T>
constexpr int gcr_unroll(int j) {
    return sizeof(T) == 4 ? (j <= 6 ? 4 : 2) : (j <= 6 ? 2 : 1);
}

__device__ __forceinline__ cpx<double> cdiv_real(cpx<double> a, double d) {
    return d > 0.0 ? cpx<double>{a.re / d, a.im / d} : cpx<double>{0.0, 0.0};
}
}  // namespace

template <typename T, int j>   // (j: directions, a template argument so that every load is unconditional)
__global__ void __launch_bounds__(kBlock)
k_gcr_multidot(const cpx<T>* W, size_t wstride, const cpx<T>* w, size_t n, GcrDev g, RedWork rw) {
    SHARED_RED;
    const int col = blockIdx.y;
    const size_t o = (size_t)col * n;
    const bool stop = g.stop[col] != 0;
    double v[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) v[q] = 0.0;
    if (!stop) GRID_STRIDE(e, n) {
        const cpx<double> we = up(w[o + e]);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i < j) {
                cpx<double> p = cjmul(up(W[(size_t)i * wstride + o + e]), we);
                v[2 * i] += p.re;
                v[2 * i + 1] += p.im;
            }
        }
    }
    write_partials<32>(v, 2 * j, rw, col, sh, tot);
}

template <typename T, int j>
__global__ void __launch_bounds__(kBlock)
k_gcr_orth(const cpx<T>* W, size_t wstride, cpx<T>* w, const cpx<T>* r, size_t n, GcrDev g, RedWork rw) {
    SHARED_RED;
    const int col = blockIdx.y;
    const bool stop = g.stop[col] != 0;
    const size_t o = (size_t)col * n;
    cpx<T> c[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        c[i] = {T(0), T(0)};
        if (i < j && !stop) {
            cpx<double> d = ld2(&g.D[(((size_t)col * g.kmax + j) * g.kmax + i) * 2]);
            cpx<double> ci = cdiv_real(d, g.nn[(size_t)col * g.kmax + i]);
            c[i] = {(T)ci.re, (T)ci.im};
        }
    }
    double v[3] = {0.0, 0.0, 0.0};
    GRID_STRIDE(e, n) {
        cpx<T> we = w[o + e];
        if (!stop && j > 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (i < j) {
                    cpx<T> Wi = W[(size_t)i * wstride + o + e];
                    we.re -= c[i].re * Wi.re - c[i].im * Wi.im;
                    we.im -= c[i].re * Wi.im + c[i].im * Wi.re;
                }
            w[o + e] = we;
        }
        const cpx<double> wd = up(we), rd = up(r[o + e]);
        v[0] += wd.re * wd.re + wd.im * wd.im;
        cpx<double> p = cjmul(wd, rd);
        v[1] += p.re;
        v[2] += p.im;
    }
    write_partials<3>(v, 3, rw, col, sh, tot);
}

__global__ void __launch_bounds__(kBlock) k_fin_gcr_orth(RedWork rw, int nb, GcrDev g, int j) {
    SHARED_RED;
    const int col = blockIdx.x;
    sum_partials<3>(3, nb, rw, col, sh, tot);
    if (threadIdx.x == 0) {
        const size_t s = (size_t)col * g.kmax + j;
        if (g.stop[col]) {
            g.nn[s] = 0.0;
            g.wr[2 * s] = 0.0;
            g.wr[2 * s + 1] = 0.0;
        } else {
            g.nn[s] = tot[0];
            g.wr[2 * s] = tot[1];
            g.wr[2 * s + 1] = tot[2];
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(kBlock)
k_gcr_rupdate(const cpx<T>* w, cpx<T>* r, cpx<T>* copy, int j, size_t n, int want_norm, GcrDev g, RedWork rw) {
    SHARED_RED;
    const int col = blockIdx.y;
    const size_t s = (size_t)col * g.kmax + j;
    const cpx<double> ad = cdiv_real(ld2(&g.wr[2 * s]), g.nn[s]);
    const cpx<T> a = {(T)ad.re, (T)ad.im};
    const size_t o = (size_t)col * n;
    double v[1] = {0.0};
    GRID_STRIDE(e, n) {
        cpx<T> re = r[o + e];
        const cpx<T> we = w[o + e];
        re.re -= a.re * we.re - a.im * we.im;
        re.im -= a.re * we.im + a.im * we.re;
        r[o + e] = re;
        if (copy) copy[o + e] = re;
        const cpx<double> rd = up(re);
        v[0] += rd.re * rd.re + rd.im * rd.im;
    }
    if (want_norm) write_partials<1>(v, 1, rw, col, sh, tot);
}

// ---- fused GCR iteration (see kernels.hpp); the direction count j is a template
// argument, so that every load of an iteration is unconditional and in flight at once
template <typename T, int j>
__global__ void __launch_bounds__(kBlock)
k_gcr_dots(const cpx<T>* W, size_t wstride, const cpx<T>* w, const cpx<T>* r, size_t n, const int* stop,
           RedWork rw) {
    SHARED_RED;
    const int col = blockIdx.y;
    const size_t o = (size_t)col * n;
    // the vectors are read whatever the stop flag says, so that no load waits for it;
    // a stopped column's sums (possibly of unwritten directions) are replaced by zeros.
    // The flag is read by a vector load (an offset the compiler cannot see is zero), which
    // completes in order with the vectors' loads instead of holding them back.
    int zoff;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zoff));
    const int sflag = stop[col + zoff];
    // layout (static indices, so the accumulators stay in registers):
    // [|w|^2, Re <w, r>, Im <w, r>, Re <W_0, w>, Im <W_0, w>, ...]
    double v[35];
#pragma unroll
    for (int q = 0; q < 35; ++q) v[q] = 0.0;
    // the entries of a thread are added in grid-stride order; U of them are loaded
    // together, so that a thread keeps U (j + 2) loads in flight (same sums, same order)
    constexpr int U = gcr_unroll<T>(j);
    auto add = [&](const cpx<T>& wt, const cpx<T>& rt, const cpx<T>* Wt) {
        const cpx<double> we = up(wt), re = up(rt);
#pragma unroll
        for (int i = 0; i < j; ++i) {
            const cpx<double> p = cjmul(up(Wt[i]), we);
            v[3 + 2 * i] += p.re;
            v[4 + 2 * i] += p.im;
        }
        v[0] += we.re * we.re + we.im * we.im;
        const cpx<double> p = cjmul(we, re);
        v[1] += p.re;
        v[2] += p.im;
    };
    {
        const size_t stride = (size_t)gridDim.x * blockDim.x;
        size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
        for (; e + (U - 1) * stride < n; e += U * stride) {
            cpx<T> wv[U], rv[U], Wv[U][j > 0 ? j : 1];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                wv[u] = w[o + e + u * stride];
                rv[u] = r[o + e + u * stride];
#pragma unroll
                for (int i = 0; i < j; ++i) Wv[u][i] = W[(size_t)i * wstride + o + e + u * stride];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) add(wv[u], rv[u], Wv[u]);
        }
        for (; e < n; e += stride) {
            cpx<T> Wt[j > 0 ? j : 1];
#pragma unroll
            for (int i = 0; i < j; ++i) Wt[i] = W[(size_t)i * wstride + o + e];
            add(w[o + e], r[o + e], Wt);
        }
    }
#pragma unroll
    for (int q = 0; q < 35; ++q) v[q] = sflag != 0 ? 0.0 : v[q];
    write_partials<35>(v, 2 * j + 3, rw, col, sh, tot);
}

template <typename T, int j>
__global__ void __launch_bounds__(kBlock)
k_gcr_fused_update(const cpx<T>* W, size_t wstride, cpx<T>* w, cpx<T>* r, cpx<T>* copy, size_t n,
                   double tol2, const int* stop_in, int* stop_out, GcrDev g) {
    const int col = blockIdx.y;
    const bool stopped = stop_in[col] != 0;
    const double* t = g.tot + (size_t)col * kGcrTot;
    const size_t kb = (size_t)col * g.kmax;
    cpx<double> c[16];
    double nnj = t[0];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        c[i] = {0.0, 0.0};
        if (i < j) {
            const cpx<double> d = {t[3 + 2 * i], t[4 + 2 * i]};
            const double nni = g.nn[kb + i];
            if (nni > 0.0) {
                c[i] = {d.re / nni, d.im / nni};
                nnj -= (d.re * d.re + d.im * d.im) / nni;
            }
        }
    }
    const cpx<double> wr = {t[1], t[2]};
    const bool live = !stopped && nnj > 0.0;
    const cpx<double> a = live ? cpx<double>{wr.re / nnj, wr.im / nnj} : cpx<double>{0.0, 0.0};
    const size_t o = (size_t)col * n;
    if (!stopped) {
        cpx<T> cc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) cc[i] = {(T)c[i].re, (T)c[i].im};
        const cpx<T> at = {(T)a.re, (T)a.im};
        // one entry: w' = w - sum c_i W_i, r -= a w', copy = r (U entries' loads issued together)
        auto step = [&](size_t i0, cpx<T> we, cpx<T> re, const cpx<T>* Wt) {
#pragma unroll
            for (int i = 0; i < j; ++i) {
                we.re -= cc[i].re * Wt[i].re - cc[i].im * Wt[i].im;
                we.im -= cc[i].re * Wt[i].im + cc[i].im * Wt[i].re;
            }
            w[i0] = we;
            re.re -= at.re * we.re - at.im * we.im;
            re.im -= at.re * we.im + at.im * we.re;
            r[i0] = re;
            if (copy) copy[i0] = re;
        };
        constexpr int U = gcr_unroll<T>(j);
        const size_t stride = (size_t)gridDim.x * blockDim.x;
        size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
        for (; e + (U - 1) * stride < n; e += U * stride) {
            cpx<T> wv[U], rv[U], Wv[U][j > 0 ? j : 1];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                wv[u] = w[o + e + u * stride];
                rv[u] = r[o + e + u * stride];
#pragma unroll
                for (int i = 0; i < j; ++i) Wv[u][i] = W[(size_t)i * wstride + o + e + u * stride];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) step(o + e + u * stride, wv[u], rv[u], Wv[u]);
        }
        for (; e < n; e += stride) {
            cpx<T> Wt[j > 0 ? j : 1];
#pragma unroll
            for (int i = 0; i < j; ++i) Wt[i] = W[(size_t)i * wstride + o + e];
            step(o + e, w[o + e], r[o + e], Wt);
        }
    } else if (copy) {
        // a column that stopped earlier in the cycle: its later directions are zero.  The
        // solution update weights them by zero coefficients, which must not meet whatever
        // the unwritten buffer holds (a non-finite word would turn 0 x into NaN), and a
        // zero direction keeps the stencil of that column finite for its tile neighbours.
        GRID_STRIDE(e, n) copy[o + e] = cpx<T>{(T)0, (T)0};
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const size_t s = kb + j;
        g.nn[s] = live ? nnj : 0.0;
        g.wr[2 * s] = live ? wr.re : 0.0;
        g.wr[2 * s + 1] = live ? wr.im : 0.0;
        for (int i = 0; i < j; ++i) {   // <W_i, w> for the back substitution
            g.D[((kb + j) * g.kmax + i) * 2] = stopped ? 0.0 : t[3 + 2 * i];
            g.D[((kb + j) * g.kmax + i) * 2 + 1] = stopped ? 0.0 : t[4 + 2 * i];
        }
        int sflag = stop_in[col];
        if (!stopped) {
            double rr = g.rr[col] - (live ? (wr.re * wr.re + wr.im * wr.im) / nnj : 0.0);
            if (rr < 0.0) rr = 0.0;
            g.rr[col] = rr;
            g.it[col] += 1;
            if (!finite(rr) || !finite(nnj)) sflag = 2;
            else if (rr <= tol2 * g.bb[col]) sflag = 1;
        }
        stop_out[col] = sflag;
    }
}

// ---- s-step GCR cycle (short cycles, Hierarchy::ss_longest: the smoother's and the coarsest
// solve's).  The cycle's minimal residual lies in r0 - span{A p : p in K_k(A, r0)}, whatever
// basis spans the Krylov space, so the directions need no inner product while they are built:
// P_0 = r0, P_{i+1} = A P_i / c - s_i P_i (the stencil's epilogue; the shifts lie inside the
// spectrum), hence A P_i = c v_i with v_i = P_{i+1} + s_i P_i.  One pass
// forms H_ab = <P_a, P_b>, one workgroup per column solves G y = b, G_il = <v_i, v_l>,
// b_i = <v_i, r0>, and one pass updates x += sum y_i P_i / c and
// P_0 = r0 - sum y_i v_i.  HBM-bound: K + 1 vectors read for the products and K + 2 read and 2
// written for the update, where a form that orthogonalises or minimises at every step reads
// j + 2 and j + 2 vectors and writes one at each step j and needs three launches there.
// 256^2 x 16 FP32, 5 steps, the fused fine A in one launch of 3 passes: 30 vector passes and 8 launches
// a cycle, against 61 and 20 for a form that minimises at every step.
namespace {
// 512 threads: half as many partials to add as 256 would leave for the same waves in flight
constexpr int kSsThreads = 512;
constexpr int ss_nq(int k) { return (k + 1) * (k + 1); }   // real sums of a (k+1)^2 Hermitian H
// complex entries of one 16-byte word, and their sum over a word
template <typename T> struct Word;
template <> struct Word<float> {
    typedef float type __attribute__((ext_vector_type(4)));
    static constexpr int E = 2;
    static __device__ __forceinline__ cpx<double> at(const type& w, int e) { return {(double)w[2 * e], (double)w[2 * e + 1]}; }
    static __device__ __forceinline__ void put(type& w, int e, cpx<double> v) { w[2 * e] = (float)v.re; w[2 * e + 1] = (float)v.im; }
};
template <> struct Word<double> {
    typedef double type __attribute__((ext_vector_type(2)));
    static constexpr int E = 1;
    static __device__ __forceinline__ cpx<double> at(const type& w, int) { return {w[0], w[1]}; }
    static __device__ __forceinline__ void put(type& w, int, cpx<double> v) { w[0] = v.re; w[1] = v.im; }
};
// offset of H_ab (a < b, two reals) behind the k + 1 diagonal entries
constexpr int ss_off(int k, int a, int b) { return (k + 1) + 2 * (a * (2 * k + 1 - a) / 2 + (b - a - 1)); }

// Sum v[0..NP) over the 64 lanes by halving: lanes that differ in one bit exchange half of their
// values each, so NP sums take NP - 1 exchanges instead of 6 NP.  The total of value i ends in
// v[0] of the lanes whose bits 0.. hold i (log2 NP of them, most significant bit of i first).
template <int NP, int BIT = 1>
__device__ __forceinline__ void reduce_scatter(double* v, int lane) {
    if constexpr (NP > 1) {
        const bool up = lane & BIT;
#pragma unroll
        for (int i = 0; i < NP / 2; ++i) {
            const double keep = up ? v[i + NP / 2] : v[i], give = up ? v[i] : v[i + NP / 2];
            v[i] = keep + __shfl_xor(give, BIT, 64);
        }
        reduce_scatter<NP / 2, BIT * 2>(v, lane);
    } else if constexpr (BIT < 64) {
        v[0] += __shfl_xor(v[0], BIT, 64);
        reduce_scatter<1, BIT * 2>(v, lane);
    }
}
// the value whose total lane `lane` holds after reduce_scatter<NP>
template <int NP, int BIT = 1>
__device__ __forceinline__ int scatter_index(int lane) {
    if constexpr (NP > 1) return ((lane & BIT) ? NP / 2 : 0) + scatter_index<NP / 2, BIT * 2>(lane);
    else return 0;
}
}  // namespace

template <typename T, int K>
__global__ void __launch_bounds__(kSsThreads) k_ss_dots(SsVecs<T> P, size_t nw, RedWork rw) {
    using W = Word<T>;
    typedef typename W::type word;
    constexpr int NQ = ss_nq(K);
    // sums in one group of a power of two up to 64, and a second small one where that fits better
    constexpr int N1 = NQ <= 4 ? 4 : (NQ <= 16 ? 16 : (NQ <= 36 ? 32 : 64));
    constexpr int N2 = NQ <= N1 ? 0 : (NQ - N1 <= 4 ? 4 : 32);
    static_assert(NQ <= N1 + N2, "two groups hold every sum");
    __shared__ double sh[kSsThreads / 64][N1 + N2];
    const int col = blockIdx.y;
    const size_t o = (size_t)col * nw;
    const word* p[K + 1];
#pragma unroll
    for (int a = 0; a <= K; ++a) p[a] = reinterpret_cast<const word*>(P.p[a]) + o;
    double v[N1 + (N2 > 0 ? N2 : 1)];
#pragma unroll
    for (int q = 0; q < N1 + N2; ++q) v[q] = 0.0;
    auto add = [&](const word* w) {
#pragma unroll
        for (int e = 0; e < W::E; ++e) {
            cpx<double> z[K + 1];
#pragma unroll
            for (int a = 0; a <= K; ++a) z[a] = W::at(w[a], e);
#pragma unroll
            for (int a = 0; a <= K; ++a) {
                v[a] = fma(z[a].re, z[a].re, v[a]);
                v[a] = fma(z[a].im, z[a].im, v[a]);
#pragma unroll
                for (int b = a + 1; b <= K; ++b) {
                    const int q = ss_off(K, a, b);
                    v[q] = fma(z[a].re, z[b].re, v[q]);
                    v[q + 1] = fma(z[a].re, z[b].im, v[q + 1]);
                    v[q] = fma(z[a].im, z[b].im, v[q]);
                    v[q + 1] = fma(-z[a].im, z[b].re, v[q + 1]);
                }
            }
        }
    };
    // U words of every vector are loaded together (bounded by the registers beside the sums)
    constexpr int U = K <= 3 ? 4 : (K <= 5 || (K == 6 && W::E == 1) ? 2 : 1);
    const size_t stride = (size_t)gridDim.x * kSsThreads;
    size_t e = (size_t)blockIdx.x * kSsThreads + threadIdx.x;
    for (; e + (U - 1) * stride < nw; e += U * stride) {
        word w[U][K + 1];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a <= K; ++a) w[u][a] = p[a][e + u * stride];
#pragma unroll
        for (int u = 0; u < U; ++u) add(w[u]);
    }
    for (; e < nw; e += stride) {
        word w[K + 1];
#pragma unroll
        for (int a = 0; a <= K; ++a) w[a] = p[a][e];
        add(w);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    reduce_scatter<N1>(v, lane);
    if (lane < N1) sh[wid][scatter_index<N1>(lane)] = v[0];
    if constexpr (N2 > 0) {
        reduce_scatter<N2>(v + N1, lane);
        if (lane < N2) sh[wid][N1 + scatter_index<N2>(lane)] = v[N1];
    }
    __syncthreads();
    // partials block by block, the sums of one block side by side
    double* part = rw.partial + (size_t)col * rw.max_q * rw.nblk + (size_t)blockIdx.x * NQ;
    for (int q = threadIdx.x; q < NQ; q += kSsThreads) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kSsThreads / 64; ++w) t += sh[w][q];
        part[q] = t;
    }
}

// One workgroup per column: wave w adds the partials of blocks w, w + 16, ... (lane = sum), then
// wave 0 factors G by Cholesky, an entry per lane.  The residual norm after step k is
// |r0|^2 - sum_{i<=k} |u_i|^2 (u = L^-1 b), so a tolerance met inside the cycle ends it at that
// step: the coefficients are those of its leading block.  Below kSsTrust of the cycle's start that
// difference is rounding; the next cycle's |P_0|^2 then decides.  A pivot within rounding of zero
// against its direction's own norm drops that direction.
// The work is small and runs once, so its time is that of fetching code and of waits in turn: unrolled
// over one row per lane it was 11 KB at 6 steps (16 KB at 8) and took 7.9 us (12.7); one entry
// per lane in rolled loops, 4 KB, and state and partials in flight together, 7.0 (9.6).
constexpr int kSsFinWaves = 16;
constexpr double kSsPivot = 1e-13;
constexpr double kSsTrust = 1e-12;
template <int K>
__global__ void __launch_bounds__(64 * kSsFinWaves) k_ss_fin(RedWork rw, int nb, GcrDev g, double tol2, SsShifts sh,
                                                            int first, SsPublish pub) {
    constexpr int NQ = ss_nq(K);
    constexpr int NR = (NQ + 63) / 64;
    __shared__ double sp[kSsFinWaves][NQ];
    __shared__ double H[NQ];
    const int col = blockIdx.x;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const double* part = rw.partial + (size_t)col * rw.max_q * rw.nblk;
    static_assert(kSsBlocks % kSsFinWaves == 0);
    constexpr int NB = kSsBlocks / kSsFinWaves;
    double pv[NR][NB];   // all of a lane's partials in flight together
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int q = r * 64 + lane < NQ ? r * 64 + lane : 0;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int b = wid + j * kSsFinWaves;
            pv[r][j] = part[(size_t)(b < nb ? b : 0) * NQ + q];
        }
    }
    // (the state is loaded with the partials, whatever `first` says, by vector loads - an offset
    // the compiler cannot see through - which it does not move behind the barriers: nothing waits in turn)
    int z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    const int stop = g.stop[col + z], iters = g.it[col + z];
    const double bbs = g.bb[col + z];
    const unsigned ctr = (pub.ctr ? pub.ctr : reinterpret_cast<const unsigned*>(g.stop))[z];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j) s += wid + j * kSsFinWaves < nb ? pv[r][j] : 0.0;
        if (r * 64 + lane < NQ) sp[wid][r * 64 + lane] = s;
    }
    __syncthreads();
    if (threadIdx.x < NQ) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kSsFinWaves; ++w) s += sp[w][threadIdx.x];
        H[threadIdx.x] = s;
    }
    __syncthreads();
    if (wid != 0) return;
    const int flag0 = first ? 0 : __builtin_amdgcn_readfirstlane(stop);
    const int it0 = first ? 0 : iters;
    const double bb0 = first ? -1.0 : bbs;
    const unsigned seq = ctr + 1u;
    double* coef = g.tot + (size_t)col * kGcrTot;   // y_i / c (2 K), then P_0's change (2 K + 2), then the live flag
    bool sane = true;
#pragma unroll
    for (int a = 0; a <= K; ++a) sane = sane && finite(H[a]);
    const double rr0 = H[0];
    const double bb = bb0 < 0.0 ? rr0 : bb0;
    int flag = flag0;
    if (flag == 0 && !sane) flag = 2;
    if (flag == 0 && (rr0 == 0.0 || (bb0 >= 0.0 && rr0 <= tol2 * bb))) flag = 1;
    auto leave = [&](int f, int it) {
        if (pub.word)
            __hip_atomic_store(pub.word + col,
                               (unsigned long long)seq << 32 | (unsigned)it << 2 | (unsigned)f,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        g.stop[col] = f;
        g.it[col] = it;
        g.bb[col] = bb;
    };
    if (flag != 0) {   // the column takes no update
        if (lane == 0) {
            coef[kGcrTot - 1] = 0.0;
            leave(flag, it0);
        }
        return;
    }
    // lane 8 i + l: entry (i, l) of G; a row's b, u and y in all of its lanes (rows and columns
    // past the last repeat it; their values go nowhere)
    auto h = [&](int a, int b) -> cpx<double> {
        const int lo = min(a, b), hi = max(a, b), q = a == b ? a : ss_off(K, lo, hi);
        const double re = H[q], im = H[q + 1];
        return {re, a == b ? 0.0 : (a < b ? im : -im)};
    };
    auto bcast = [](double x, int l) {   // lane l's value, the same for the whole wave
        const int lo = __builtin_amdgcn_readlane(__double2loint(x), l), hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
        return __hiloint2double(hi, lo);
    };
    auto from = [](cpx<double> z, int l) -> cpx<double> { return {__shfl(z.re, l), __shfl(z.im, l)}; };
    const int row = lane >> 3, colm = lane & 7;
    const int i = row < K ? row : K - 1, l = colm < K ? colm : K - 1;
    double si = sh.s[0], sl = sh.s[0];   // (selects: the arguments are not indexed by lane)
#pragma unroll
    for (int j = 1; j < K; ++j) {
        si = i == j ? sh.s[j] : si;
        sl = l == j ? sh.s[j] : sl;
    }
    cpx<double> G = h(i + 1, l + 1) + sl * h(i + 1, l) + si * h(i, l + 1) + si * sl * h(i, l);
    cpx<double> bi = h(i + 1, 0) + si * h(i, 0);
    const double dg = G.re;
    cpx<double> L = {0.0, 0.0}, u = {0.0, 0.0};
    double rr = rr0, inv = 0.0;
    int kend = 0;
#pragma unroll 1
    for (int k = 0; k < K && flag == 0; ++k) {   // (uniform)
        const double d = bcast(G.re, 9 * k), d0 = bcast(dg, 9 * k);
        const double ik = d > kSsPivot * d0 && finite(d) ? rsqrt(d) : 0.0;
        const cpx<double> uk = {bcast(bi.re, 8 * k) * ik, bcast(bi.im, 8 * k) * ik};
        cpx<double> lk = from(G, (i << 3) + k), ll = from(G, (l << 3) + k);   // L_ik and L_lk
        lk = {lk.re * ik, lk.im * ik};
        ll = {ll.re * ik, ll.im * ik};
        if (l == k) L = lk;
        if (i == k) { u = uk; inv = ik; }
        G.re -= lk.re * ll.re + lk.im * ll.im;   // G_il -= L_ik conj(L_lk)
        G.im -= lk.im * ll.re - lk.re * ll.im;
        bi.re -= lk.re * uk.re - lk.im * uk.im;
        bi.im -= lk.re * uk.im + lk.im * uk.re;
        rr -= uk.re * uk.re + uk.im * uk.im;
        kend = k + 1;
        if (!finite(rr)) flag = 2;
        else if (rr <= tol2 * bb && rr > kSsTrust * rr0) flag = 1;
    }
    cpx<double> y = {0.0, 0.0};
    if (flag != 2) {
#pragma unroll 1
        for (int k = kend - 1; k >= 0; --k) {   // L^H y = u over the steps taken
            const double ik = bcast(inv, 8 * k);
            const cpx<double> yk = {bcast(u.re, 8 * k) * ik, bcast(u.im, 8 * k) * ik};
            const cpx<double> t = cjmul(from(L, (k << 3) + i), yk);
            if (i == k) y = yk;
            u.re -= t.re;
            u.im -= t.im;
        }
    }
    const cpx<double> up = from(y, i > 0 ? (i - 1) << 3 : 0);
    const cpx<double> prev = i > 0 ? up : cpx<double>{0.0, 0.0};
    if (row < K && colm == 0) {
        coef[2 * i] = y.re * sh.inv_c;
        coef[2 * i + 1] = y.im * sh.inv_c;
        double* e = coef + 2 * K;
        e[2 * i] = -(si * y.re + prev.re);
        e[2 * i + 1] = -(si * y.im + prev.im);
        if (i == K - 1) {
            e[2 * K] = -y.re;
            e[2 * K + 1] = -y.im;
        }
    }
    if (lane == 0) {
        coef[kGcrTot - 1] = flag == 2 ? 0.0 : 1.0;
        leave(flag, it0 + kend);
    }
}

template <typename T, int K>
__global__ void __launch_bounds__(kBlock) k_ss_update(SsVecs<T> P, cpx<T>* x, size_t nw, GcrDev g, unsigned* ctr) {
    using W = Word<T>;
    typedef typename W::type word;
    const int col = blockIdx.y;
    if (ctr && blockIdx.x == 0 && col == 0 && threadIdx.x == 0) *ctr += 1u;   // (no other workgroup reads it)
    const double* coef = g.tot + (size_t)col * kGcrTot;
    cpx<double> y[K], d[K + 1];
#pragma unroll
    for (int k = 0; k < K; ++k) y[k] = ld2(coef + 2 * k);
#pragma unroll
    for (int k = 0; k <= K; ++k) d[k] = ld2(coef + 2 * K + 2 * k);
    if (coef[kGcrTot - 1] == 0.0) return;   // a column that takes no update (its vectors may be anything)
    const size_t o = (size_t)col * nw;
    word* xw = reinterpret_cast<word*>(x) + o;
    word* p0 = reinterpret_cast<word*>(P.p[0]) + o;
    auto step = [&](size_t e, const word* w, word xv) {
        word r;
#pragma unroll
        for (int c = 0; c < W::E; ++c) {
            cpx<double> xa = W::at(xv, c), ra = W::at(w[0], c);
#pragma unroll
            for (int k = 0; k <= K; ++k) {
                const cpx<double> z = W::at(w[k], c);
                if (k < K) {
                    xa.re = fma(y[k].re, z.re, xa.re);
                    xa.im = fma(y[k].re, z.im, xa.im);
                    xa.re = fma(-y[k].im, z.im, xa.re);
                    xa.im = fma(y[k].im, z.re, xa.im);
                }
                ra.re = fma(d[k].re, z.re, ra.re);
                ra.im = fma(d[k].re, z.im, ra.im);
                ra.re = fma(-d[k].im, z.im, ra.re);
                ra.im = fma(d[k].im, z.re, ra.im);
            }
            W::put(xv, c, xa);
            W::put(r, c, ra);
        }
        xw[e] = xv;
        p0[e] = r;
    };
    constexpr int U = K <= 6 ? 2 : 1;
    const size_t stride = (size_t)gridDim.x * kBlock;
    size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    for (; e + (U - 1) * stride < nw; e += U * stride) {
        word w[U][K + 1], xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int k = 0; k <= K; ++k) w[u][k] = reinterpret_cast<const word*>(P.p[k])[o + e + u * stride];
            xv[u] = xw[e + u * stride];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) step(e + u * stride, w[u], xv[u]);
    }
    for (; e < nw; e += stride) {
        word w[K + 1];
#pragma unroll
        for (int k = 0; k <= K; ++k) w[k] = reinterpret_cast<const word*>(P.p[k])[o + e];
        step(e, w, xw[e]);
    }
}

// start of a device-driven s-step solve: P_0 = b, x = 0, and the columns' state (|b|^2 not known yet)
template <typename T>
__global__ void k_ss_begin(const cpx<T>* b, cpx<T>* P0, cpx<T>* x, size_t n, int ncol, GcrDev g) {
    if (blockIdx.x == 0)
        for (int c = threadIdx.x; c < ncol; c += blockDim.x) {
            g.stop[c] = 0;
            g.it[c] = 0;
            g.bb[c] = -1.0;
        }
    GRID_STRIDE(i, n) {
        P0[i] = b[i];
        x[i] = cpx<T>{T(0), T(0)};
    }
}

// restart of the device-driven GCR on the recursive residual: the next first
// direction is r, and the stop flags of the last step move to g.stop
template <typename T>
__global__ void k_gcr_restart(const cpx<T>* r, cpx<T>* P0, size_t n, const int* stop_src, int* stop, int ncol) {
    if (blockIdx.x == 0 && stop_src != stop)
        for (int c = threadIdx.x; c < ncol; c += blockDim.x) stop[c] = stop_src[c];
    GRID_STRIDE(i, n) P0[i] = r[i];
}

__global__ void k_gcr_dev_init(int ncol, GcrDev g) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncol) return;
    const double b = g.rr[c];
    g.bb[c] = b;
    g.it[c] = 0;
    g.stop[c] = finite(b) ? (b == 0.0 ? 1 : 0) : 2;
}

// back substitution gam_j = (wr_j - sum_{l>j} D[l][j] gam_l) / nn_j, from arrays laid out
// as in GcrDev (row stride ds of D); shared by the one-thread kernel and the x-update
__device__ __forceinline__ void gcr_back_substitute(int k, const double* wr, const double* nn, const double* D,
                                                    size_t ds, double* gam) {
    for (int j = k - 1; j >= 0; --j) {
        cpx<double> gj = cdiv_real(ld2(&wr[2 * j]), nn[j]);
        for (int l = j + 1; l < k; ++l) {
            // beta_{j l} = <w_j, A p_l> / |w_j|^2
            cpx<double> bjl = cdiv_real(ld2(&D[(l * ds + j) * 2]), nn[j]);
            cpx<double> gl = ld2(&gam[2 * l]);
            cpx<double> t = cmul(bjl, gl);
            gj.re -= t.re;
            gj.im -= t.im;
        }
        gam[2 * j] = gj.re;
        gam[2 * j + 1] = gj.im;
    }
}

__global__ void k_gcr_solve(int k, int ncol, GcrDev g) {
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= ncol) return;
    const size_t b = (size_t)col * g.kmax;
    gcr_back_substitute(k, g.wr + 2 * b, g.nn + b, g.D + b * g.kmax * 2, (size_t)g.kmax, g.gam + 2 * b);
}

// (the direction count K is a template argument, as in the fused GCR kernels: with a
// run-time count every direction's load sat behind its own branch and waited there)
template <typename T, typename Tx, int K>
__global__ void k_gcr_xupdate(const cpx<T>* P, size_t pstride, cpx<Tx>* x, size_t n, int accumulate, GcrDev g,
                              int solve, const cpx<T>* rsrc, cpx<T>* p0dst, const int* stop_src, int ncol) {
    constexpr int k = K;
    const int col = blockIdx.y;
    const size_t o = (size_t)col * n;
    const double* gam = g.gam + 2 * (size_t)col * g.kmax;
    __shared__ double sD[16 * 16 * 2], snn[16], swr[32], sgam[32];
    if (solve) {
        // every block solves the small triangular system itself (the same arithmetic in
        // the same order as the one-thread kernel): the entries are loaded in parallel
        // into LDS, one thread substitutes, block 0 stores gam
        const size_t b = (size_t)col * g.kmax;
        for (int t = threadIdx.x; t < k * k; t += blockDim.x) {
            const int l = t / k, j = t - l * k;
            sD[(l * 16 + j) * 2] = g.D[((b + l) * g.kmax + j) * 2];
            sD[(l * 16 + j) * 2 + 1] = g.D[((b + l) * g.kmax + j) * 2 + 1];
        }
        if (threadIdx.x < k) {
            snn[threadIdx.x] = g.nn[b + threadIdx.x];
            swr[2 * threadIdx.x] = g.wr[2 * (b + threadIdx.x)];
            swr[2 * threadIdx.x + 1] = g.wr[2 * (b + threadIdx.x) + 1];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            gcr_back_substitute(k, swr, snn, sD, 16, sgam);
            if (blockIdx.x == 0)
                for (int i = 0; i < 2 * k; ++i) g.gam[2 * b + i] = sgam[i];
        }
        __syncthreads();
        gam = sgam;
    }
    cpx<double> c[K > 0 ? K : 1];
#pragma unroll
    for (int i = 0; i < K; ++i) c[i] = cpx<double>{gam[2 * i], gam[2 * i + 1]};
    if (stop_src && stop_src != g.stop && blockIdx.x == 0 && blockIdx.y == 0)
        for (int cc = threadIdx.x; cc < ncol; cc += blockDim.x) g.stop[cc] = stop_src[cc];
    GRID_STRIDE(e, n) {
        cpx<double> acc = {0.0, 0.0};
        if (accumulate) acc = {(double)x[o + e].re, (double)x[o + e].im};
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const cpx<double> p = up(P[(size_t)i * pstride + o + e]);
            acc.re += c[i].re * p.re - c[i].im * p.im;
            acc.im += c[i].re * p.im + c[i].im * p.re;
        }
        x[o + e] = {(Tx)acc.re, (Tx)acc.im};
        // restart: the residual becomes the first direction (after P_0 was read above)
        if (p0dst) p0dst[o + e] = rsrc[o + e];
    }
}

template <typename T>
hipError_t gcr_multidot(const cpx<T>* W, size_t wstride, int j, const cpx<T>* w, size_t n, int ncol,
                        const GcrDev& g, const RedWork& rw, hipStream_t st) {
    if (j <= 0) return hipSuccess;
    if (j > 16) return hipErrorInvalidValue;
    dim3 grid = red_grid(n, ncol, rw);
    with_j(j, [&](auto jc) {
        hipLaunchKernelGGL((k_gcr_multidot<T, decltype(jc)::value>), grid, dim3(kBlock), 0, st, W, wstride, w, n, g, rw);
    }, std::make_integer_sequence<int, 17>{});
    hipLaunchKernelGGL(k_fin_store_q, dim3(2 * j, ncol), dim3(kBlock), 0, st, rw, (int)grid.x,
                       g.D + (size_t)j * g.kmax * 2, (size_t)g.kmax * g.kmax * 2);
    return hipGetLastError();
}
template <typename T>
hipError_t gcr_orth(const cpx<T>* W, size_t wstride, int j, cpx<T>* w, const cpx<T>* r, size_t n,
                    int ncol, const GcrDev& g, const RedWork& rw, hipStream_t st) {
    if (j > 16) return hipErrorInvalidValue;
    if (j < 0) return hipErrorInvalidValue;
    dim3 grid = red_grid(n, ncol, rw);
    with_j(j, [&](auto jc) {
        hipLaunchKernelGGL((k_gcr_orth<T, decltype(jc)::value>), grid, dim3(kBlock), 0, st, W, wstride, w, r, n, g, rw);
    }, std::make_integer_sequence<int, 17>{});
    hipLaunchKernelGGL(k_fin_gcr_orth, dim3(ncol), dim3(kBlock), 0, st, rw, (int)grid.x, g, j);
    return hipGetLastError();
}
template <typename T>
hipError_t gcr_rupdate(const cpx<T>* w, cpx<T>* r, cpx<T>* copy, int j, size_t n, int ncol,
                       bool want_norm, const GcrDev& g, const RedWork& rw, hipStream_t st) {
    dim3 grid = want_norm ? red_grid(n, ncol, rw) : ew_grid(n, ncol);
    hipLaunchKernelGGL(k_gcr_rupdate<T>, grid, dim3(kBlock), 0, st, w, r, copy, j, n, want_norm ? 1 : 0, g, rw);
    if (want_norm)
        hipLaunchKernelGGL(k_fin_store, dim3(ncol), dim3(kBlock), 0, st, rw, 1, (int)grid.x, g.rr, (size_t)1);
    return hipGetLastError();
}
template <typename T>
hipError_t gcr_fused_step(const cpx<T>* W, size_t wstride, int j, cpx<T>* w, cpx<T>* r, cpx<T>* copy, size_t n,
                          int ncol, double tol2, const int* stop_in, int* stop_out, const GcrDev& g,
                          const RedWork& rw, hipStream_t st) {
    if (j < 0 || j > 15 || 2 * j + 3 > kGcrTot || 2 * j + 3 > rw.max_q) return hipErrorInvalidValue;
    const dim3 grid = red_grid(n, ncol, rw);
    auto launch = [&](auto jc) {
        constexpr int J = decltype(jc)::value;
        hipLaunchKernelGGL((k_gcr_dots<T, J>), grid, dim3(kBlock), 0, st, W, wstride, w, r, n, stop_in, rw);
        hipLaunchKernelGGL(k_fin_store_q1, dim3(2 * J + 3, ncol), dim3(64), 0, st, rw, (int)grid.x, g.tot,
                           (size_t)kGcrTot);
        hipLaunchKernelGGL((k_gcr_fused_update<T, J>), ew_grid(n, ncol), dim3(kBlock), 0, st, W, wstride, w, r,
                           copy, n, tol2, stop_in, stop_out, g);
    };
    with_j(j, launch, std::make_integer_sequence<int, 16>{});
    return hipGetLastError();
}
template <typename T>
hipError_t ss_begin(const cpx<T>* b, cpx<T>* P0, cpx<T>* x, size_t n, int ncol, const GcrDev& g, hipStream_t st) {
    hipLaunchKernelGGL(k_ss_begin<T>, ew_grid(n * ncol, 1), dim3(kBlock), 0, st, b, P0, x, n * ncol, ncol, g);
    return hipGetLastError();
}
template <typename T>
hipError_t ss_finish(const SsVecs<T>& P, int k, cpx<T>* x, size_t n, int ncol, const SsShifts& sh, double tol2, bool first,
                     const GcrDev& g, const RedWork& rw, hipStream_t st, const SsPublish& pub) {
    if (k < 1 || k > kSsMax || (pub.word && !pub.ctr) || 4 * k + 3 > kGcrTot || n % Word<T>::E) return hipErrorInvalidValue;
    const size_t nw = n / Word<T>::E;
    // blocks per column: two words per thread at least, one workgroup per CU over all columns
    // (a block's sums cost as much as streaming several words, and one workgroup adds them all)
    long long nb = (long long)((nw + 2 * kSsThreads - 1) / (2 * kSsThreads));
    nb = std::min<long long>(nb, std::max(kSsBlocks / ncol, 32));
    nb = std::max<long long>(std::min<long long>(nb, (long long)rw.max_q * rw.nblk / ss_nq(k)), 1);
    auto launch = [&](auto kc) {
        constexpr int K = decltype(kc)::value + 1;
        hipLaunchKernelGGL((k_ss_dots<T, K>), dim3((unsigned)nb, ncol), dim3(kSsThreads), 0, st, P, nw, rw);
        hipLaunchKernelGGL(k_ss_fin<K>, dim3(ncol), dim3(64 * kSsFinWaves), 0, st, rw, (int)nb, g, tol2, sh,
                           first ? 1 : 0, pub);
        hipLaunchKernelGGL((k_ss_update<T, K>), ew_grid(nw, ncol), dim3(kBlock), 0, st, P, x, nw, g,
                           pub.word ? pub.ctr : nullptr);
    };
    with_j(k - 1, launch, std::make_integer_sequence<int, kSsMax>{});
    return hipGetLastError();
}
template <typename T>
hipError_t gcr_restart(const cpx<T>* r, cpx<T>* P0, size_t n, int ncol, const int* stop_src, const GcrDev& g,
                       hipStream_t st) {
    hipLaunchKernelGGL(k_gcr_restart<T>, ew_grid(n * ncol, 1), dim3(kBlock), 0, st, r, P0, n * ncol, stop_src, g.stop,
                       ncol);
    return hipGetLastError();
}
hipError_t gcr_dev_init(int ncol, const GcrDev& g, hipStream_t st) {
    hipLaunchKernelGGL(k_gcr_dev_init, dim3(grid_for(ncol, 64)), dim3(64), 0, st, ncol, g);
    return hipGetLastError();
}
hipError_t gcr_solve(int k, int ncol, const GcrDev& g, hipStream_t st) {
    hipLaunchKernelGGL(k_gcr_solve, dim3(grid_for(ncol, 64)), dim3(64), 0, st, k, ncol, g);
    return hipGetLastError();
}
template <typename T, typename Tx>
void launch_xupdate(const cpx<T>* P, size_t pstride, int k, cpx<Tx>* x, size_t n, int ncol, bool accumulate,
                    const GcrDev& g, int solve, const cpx<T>* rsrc, cpx<T>* p0dst, const int* stop_src,
                    hipStream_t st) {
    with_j(k, [&](auto kc) {
        hipLaunchKernelGGL((k_gcr_xupdate<T, Tx, decltype(kc)::value>), ew_grid(n, ncol), dim3(kBlock), 0, st, P,
                           pstride, x, n, accumulate ? 1 : 0, g, solve, rsrc, p0dst, stop_src, ncol);
    }, std::make_integer_sequence<int, 17>{});
}
template <typename T, typename Tx>
hipError_t gcr_xupdate(const cpx<T>* P, size_t pstride, int k, cpx<Tx>* x, size_t n, int ncol,
                       bool accumulate, const GcrDev& g, hipStream_t st) {
    if (k < 0 || k > 16) return hipErrorInvalidValue;
    launch_xupdate<T, Tx>(P, pstride, k, x, n, ncol, accumulate, g, 0, nullptr, nullptr, nullptr, st);
    return hipGetLastError();
}
template <typename T, typename Tx>
hipError_t gcr_solve_xupdate(const cpx<T>* P, size_t pstride, int k, cpx<Tx>* x, size_t n, int ncol,
                             bool accumulate, const GcrDev& g, hipStream_t st) {
    if (k < 0 || k > 16) return hipErrorInvalidValue;
    // (the substitution is serial in every block: beyond 8 directions the separate
    // one-thread kernel is cheaper, measured with 16)
    if (k > 8) {
        if (hipError_t e = gcr_solve(k, ncol, g, st)) return e;
        return gcr_xupdate<T, Tx>(P, pstride, k, x, n, ncol, accumulate, g, st);
    }
    launch_xupdate<T, Tx>(P, pstride, k, x, n, ncol, accumulate, g, 1, nullptr, nullptr, nullptr, st);
    return hipGetLastError();
}
template <typename T>
hipError_t gcr_solve_xupdate_restart(cpx<T>* P, size_t pstride, int k, cpx<T>* x, size_t n, int ncol, const cpx<T>* r,
                                     const int* stop_src, const GcrDev& g, hipStream_t st) {
    if (k < 0 || k > 16) return hipErrorInvalidValue;
    if (k > 8) {
        if (hipError_t e = gcr_solve_xupdate<T, T>(P, pstride, k, x, n, ncol, true, g, st)) return e;
        return gcr_restart<T>(r, P, n, ncol, stop_src, g, st);
    }
    launch_xupdate<T, T>(P, pstride, k, x, n, ncol, true, g, 1, r, P, stop_src, st);
    return hipGetLastError();
}

// ------------------------------------------------------------ finiteness check
template <typename T>
__global__ void k_check_finite(const cpx<T>* x, size_t n, int* flag) {
    bool bad = false;
    GRID_STRIDE(i, n) {
        cpx<T> a = x[i];
        if (isnan(a.re) || isnan(a.im) || isinf(a.re) || isinf(a.im)) bad = true;
    }
    if (bad) flag[0] = 1;
}
template <typename T>
hipError_t check_finite(const cpx<T>* x, size_t n, int* flag, hipStream_t st) {
    hipLaunchKernelGGL(k_check_finite<T>, ew_grid(n, 1), dim3(kBlock), 0, st, x, n, flag);
    return hipGetLastError();
}

// ------------------------------------------------------------ instantiations
#define INST_T(T)                                                                                       \
    template hipError_t vzero<T>(cpx<T>*, size_t, hipStream_t);                                         \
    template hipError_t vsub<T>(const cpx<T>*, const cpx<T>*, cpx<T>*, size_t, hipStream_t);            \
    template hipError_t norm2<T>(const cpx<T>*, size_t, int, double*, const RedWork&, hipStream_t);     \
    template hipError_t cdot<T>(const cpx<T>*, const cpx<T>*, size_t, int, double*, const RedWork&, hipStream_t); \
    template hipError_t cg_init<T>(const cpx<T>*, size_t, int, CgScal*, double, const RedWork&, hipStream_t); \
    template hipError_t cg_alpha<T>(const cpx<T>*, size_t, int, CgScal*, const RedWork&, hipStream_t); \
    template hipError_t cg_update_xr<T>(cpx<T>*, cpx<T>*, const cpx<T>*, const cpx<T>*, size_t, int, const CgScal*, hipStream_t); \
    template hipError_t cg_beta<T>(const cpx<T>*, size_t, int, CgScal*, int, const RedWork&, hipStream_t); \
    template hipError_t cg_update_p<T>(cpx<T>*, const cpx<T>*, size_t, int, const CgScal*, hipStream_t); \
    template hipError_t cgnr_xr<T>(cpx<T>*, cpx<T>*, const cpx<T>*, const cpx<T>*, size_t, int, const CgScal*, double*, const double*, size_t, int, hipStream_t); \
    template hipError_t cgnr_p<T>(cpx<T>*, const cpx<T>*, size_t, int, int, const double*, CgScal*, const double*, size_t, int, hipStream_t); \
    template hipError_t norm2_partials<T>(const cpx<T>*, size_t, int, const CgScal*, double*, size_t, int*, hipStream_t); \
    template hipError_t gcr_multidot<T>(const cpx<T>*, size_t, int, const cpx<T>*, size_t, int, const GcrDev&, const RedWork&, hipStream_t); \
    template hipError_t gcr_orth<T>(const cpx<T>*, size_t, int, cpx<T>*, const cpx<T>*, size_t, int, const GcrDev&, const RedWork&, hipStream_t); \
    template hipError_t gcr_rupdate<T>(const cpx<T>*, cpx<T>*, cpx<T>*, int, size_t, int, bool, const GcrDev&, const RedWork&, hipStream_t); \
    template hipError_t gcr_fused_step<T>(const cpx<T>*, size_t, int, cpx<T>*, cpx<T>*, cpx<T>*, size_t, int, double, const int*, int*, const GcrDev&, const RedWork&, hipStream_t); \
    template hipError_t gcr_restart<T>(const cpx<T>*, cpx<T>*, size_t, int, const int*, const GcrDev&, hipStream_t); \
    template hipError_t check_finite<T>(const cpx<T>*, size_t, int*, hipStream_t);

INST_T(float)
INST_T(double)

template hipError_t vconvert<double, float>(const cpx<double>*, cpx<float>*, size_t, hipStream_t);
template hipError_t vconvert<float, double>(const cpx<float>*, cpx<double>*, size_t, hipStream_t);
template hipError_t vconvert<double, double>(const cpx<double>*, cpx<double>*, size_t, hipStream_t);
template hipError_t vconvert<float, float>(const cpx<float>*, cpx<float>*, size_t, hipStream_t);
template hipError_t vadd<float, double>(const cpx<float>*, cpx<double>*, size_t, hipStream_t);
template hipError_t vadd<double, double>(const cpx<double>*, cpx<double>*, size_t, hipStream_t);
template hipError_t vadd<float, float>(const cpx<float>*, cpx<float>*, size_t, hipStream_t);
template hipError_t gcr_xupdate<float, float>(const cpx<float>*, size_t, int, cpx<float>*, size_t, int, bool, const GcrDev&, hipStream_t);
template hipError_t gcr_xupdate<double, double>(const cpx<double>*, size_t, int, cpx<double>*, size_t, int, bool, const GcrDev&, hipStream_t);
template hipError_t gcr_xupdate<float, double>(const cpx<float>*, size_t, int, cpx<double>*, size_t, int, bool, const GcrDev&, hipStream_t);
template hipError_t gcr_solve_xupdate<float, float>(const cpx<float>*, size_t, int, cpx<float>*, size_t, int, bool, const GcrDev&, hipStream_t);
template hipError_t gcr_solve_xupdate<double, double>(const cpx<double>*, size_t, int, cpx<double>*, size_t, int, bool, const GcrDev&, hipStream_t);
template hipError_t ss_begin<float>(const cpx<float>*, cpx<float>*, cpx<float>*, size_t, int, const GcrDev&, hipStream_t);
template hipError_t ss_begin<double>(const cpx<double>*, cpx<double>*, cpx<double>*, size_t, int, const GcrDev&, hipStream_t);
template hipError_t ss_finish<float>(const SsVecs<float>&, int, cpx<float>*, size_t, int, const SsShifts&, double, bool, const GcrDev&, const RedWork&, hipStream_t, const SsPublish&);
template hipError_t ss_finish<double>(const SsVecs<double>&, int, cpx<double>*, size_t, int, const SsShifts&, double, bool, const GcrDev&, const RedWork&, hipStream_t, const SsPublish&);
template hipError_t gcr_solve_xupdate_restart<float>(cpx<float>*, size_t, int, cpx<float>*, size_t, int, const cpx<float>*, const int*, const GcrDev&, hipStream_t);
template hipError_t gcr_solve_xupdate_restart<double>(cpx<double>*, size_t, int, cpx<double>*, size_t, int, const cpx<double>*, const int*, const GcrDev&, hipStream_t);

}  // namespace dwf
