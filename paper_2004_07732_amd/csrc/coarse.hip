// Coarse-level operator: the Galerkin kernel hat-D_W = P^dagger D_W P in
// stencil form (Sec. 2.3) and the coarse domain-wall operator of
// eq. coarsenDW built on it:
//   hat-D_DW(m) psi_s = (hat-D_W(M5) + 1) psi_s + hatP_- psi_{s+1} + hatP_+ psi_{s-1}
// with hatP_pm = (1 pm sigma_3)/2 and the -m corners, and
//   hat-D_W psi(x) = X(x) psi(x) + sum_h Y_h(x) psi(x + h)   (X includes M5 via a shift).
// The adjoint uses sigma_3-hermiticity of the Galerkin kernel
// (gamma_5 P = P sigma_3): hat-D_W^dagger = sigma_3 hat-D_W sigma_3.
//
// Two VALU kernels.  n >= 16 (coarse_block_kernel): five wavefronts per coarse site, one per
// block of the stencil, over a tile of (right-hand side, slice) columns.  n < 16
// (coarse_kernel): one wavefront per (coarse site, column), all five blocks.  Links may be
// stored in FP64, FP32, BF16 or FP16; the latter three are multiplied in FP32.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace dwf {

// One wavefront per (coarse site, column).  The five neighbour
// vectors of all coarse slices are staged in LDS (converted to the arithmetic
// type, sigma_3 applied for the adjoint); lane i owns output row i and a
// stride of the 5n inner index, reading links blk[k][i] that are contiguous
// across lanes.  Each link element is read once per pass of eight coarse
// slices (once per apply for L-hat_s <= 8) and used for every slice of it.
template <typename L, typename T, int N, bool DAG, bool WIL>
__global__ void __launch_bounds__(256)
coarse_kernel(const L* __restrict__ links, const cpx<T>* __restrict__ in, cpx<T>* __restrict__ out,
              const int* __restrict__ skip, int skip_stride, int Lx, int Ly, int Ls, int nsites,
              typename acc_of<L>::type cdiag, typename acc_of<L>::type mwrap, const cpx<T>* __restrict__ eb, T ealpha,
              T ebeta) {
    using A = typename acc_of<L>::type;
    constexpr int P = (N <= 64) ? (64 / N) : 1;   // partitions of the inner index
    constexpr int MAXS = 8;                       // slices accumulated per pass
    constexpr int H = N / 2;
    extern __shared__ unsigned char smem_raw[];
    const int wpb = blockDim.x >> 6;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int site = (int)xcd_block(blockIdx.x, gridDim.x) * wpb + wave;
    const int col = blockIdx.y;
    // per wave: the five staged neighbour vectors; the partition sums of a pass (P > 1)
    // follow them, or with a single pass overwrite them
    cpx<A>* my = reinterpret_cast<cpx<A>*>(smem_raw) + (size_t)wave * coarse_lds_per_wave(N, Ls);
    cpx<A>* scr = (Ls <= MAXS) ? my : my + (size_t)5 * N * Ls;
    const bool valid = (site < nsites) && !(skip && skip[(size_t)col * skip_stride]);

    int nb[5] = {0, 0, 0, 0, 0};
    const cpx<T>* src = in + (size_t)col * Ls * nsites * N;
    cpx<T>* dst = out + (size_t)col * Ls * nsites * N;
    if (valid) {
        const int x = site % Lx, y = site / Lx;
        const int xp = (x + 1 == Lx) ? 0 : x + 1, xm = (x == 0) ? Lx - 1 : x - 1;
        const int yp = (y + 1 == Ly) ? 0 : y + 1, ym = (y == 0) ? Ly - 1 : y - 1;
        nb[0] = site; nb[1] = y * Lx + xp; nb[2] = y * Lx + xm; nb[3] = yp * Lx + x; nb[4] = ym * Lx + x;
        for (int e = lane; e < 5 * Ls * N; e += 64) {
            const int d = e / (Ls * N), rem = e - d * Ls * N;
            const int s = rem / N, k = rem - s * N;
            cpx<T> v = src[((size_t)s * nsites + nb[d]) * N + k];
            A re = (A)v.re, im = (A)v.im;
            if (DAG && k >= H) { re = -re; im = -im; }
            my[e] = {re, im};
        }
    }
    __syncthreads();

    const int i = lane % N;
    const int part = lane / N;
    const L* lk = links + (size_t)site * 5 * N * N;
    // slices in passes of MAXS (the accumulators stay in registers); every wave
    // takes every pass, so the barriers are uniform
    for (int s0 = 0; s0 < Ls; s0 += MAXS) {
        cpx<A> acc[MAXS];
#pragma unroll
        for (int s = 0; s < MAXS; ++s) acc[s] = {A(0), A(0)};
        if (valid && part < P) {
            for (int kk = part; kk < 5 * N; kk += P) {
                const int d = kk / N, k = kk - d * N;
                const cpx<A> l = load_link(lk, (size_t)kk * N + i);
                const cpx<A>* pv = my + (size_t)d * Ls * N + (size_t)s0 * N + k;
#pragma unroll
                for (int s = 0; s < MAXS; ++s)
                    if (s0 + s < Ls) cfma(acc[s], l, pv[(size_t)s * N]);
            }
        }
        // partition sums in a fixed order
        if (P > 1) {
            if (Ls <= MAXS) __syncthreads();   // (they overwrite the staged vectors)
            if (valid && part < P) {
#pragma unroll
                for (int s = 0; s < MAXS; ++s)
                    if (s0 + s < Ls) scr[(size_t)s * 64 + part * N + i] = acc[s];
            }
            __syncthreads();
        }
        if (valid && part == 0) {
#pragma unroll
            for (int s1 = 0; s1 < MAXS; ++s1) {
                const int s = s0 + s1;
                if (s >= Ls) break;
                cpx<A> v = {A(0), A(0)};
                if (P > 1) {
                    for (int p = 0; p < P; ++p) v = v + scr[(size_t)s1 * 64 + p * N + i];
                } else {
                    v = acc[s1];
                }
                if (DAG && i >= H) { v.re = -v.re; v.im = -v.im; }
                const cpx<T> c = src[((size_t)s * nsites + site) * N + i];
                v.re += cdiag * (A)c.re;
                v.im += cdiag * (A)c.im;
                if (!WIL) {
                    const bool minus = (i >= H);
                    // non-adjoint: hatP_- psi_{s+1} + hatP_+ psi_{s-1}; adjoint swaps
                    const bool from_up = DAG ? !minus : minus;
                    int so;
                    A f = A(1);
                    if (from_up) {
                        so = s + 1;
                        if (so == Ls) { so = 0; f = mwrap; }
                    } else {
                        so = s - 1;
                        if (so < 0) { so = Ls - 1; f = mwrap; }
                    }
                    const cpx<T> h = src[((size_t)so * nsites + site) * N + i];
                    v.re += f * (A)h.re;
                    v.im += f * (A)h.im;
                }
                const size_t oi = ((size_t)s * nsites + site) * N + i;
                cpx<T> o = {(T)v.re, (T)v.im};
                if (eb) {   // beta eb + alpha (operator in)
                    const cpx<T> b = eb[(size_t)col * Ls * nsites * N + oi];
                    o = {ealpha * o.re + ebeta * b.re, ealpha * o.im + ebeta * b.im};
                }
                dst[oi] = o;
            }
        }
        if (P > 1) __syncthreads();   // scr is rewritten by the next pass
    }
}

// ------------------------------------------------------------ one wavefront per stencil block
// Bound by the link bytes (5 n^2 entries a site) in L2 and Infinity Cache and by their latency.
// Wave d of a site's workgroup owns block d, so a site's links are in flight on five waves at
// once (one wave per site and column left one wave per SIMD at 32^2 sites: 42 us for 84 MB of
// FP64 links at n = 32, 4 slices).  A lane holds RT rows of the block at every KG-th inner index:
// row i = rt RI + i', column k = ks KG + kq, with the index that is contiguous in memory on the
// consecutive lanes, 128 bytes at a time in FP64, KC inner steps ahead of their use; every column
// tile reads them again (from L2 after the first).  Only the site term and the forward hops are read: the backward hop of a site is
// the sigma_3-adjoint of its neighbour's forward hop (gamma_5-hermiticity and a chirality-keeping
// prolongator), which that neighbour's own wave has just read into L2 on the same XCD.
// A tile whose columns have all stopped costs the flags and the first links.
// A wave stages its own neighbour's vectors in LDS, [k][column], sums over its kq lanes by
// halving exchanges and leaves its part there; after one barrier a thread per output adds the
// five parts in order with the site-local terms.

// v[0..NV) summed over KG lanes (lane bits from SH up): halving exchanges while the count is
// even, then butterflies; returns the first index of the values this lane ends with and their
// count in `left`, and whether it is the lane that writes them
template <typename A, int NV, int KG, int SH>
__device__ __forceinline__ int lane_reduce(A* v, int lane, bool& writes) {
    int base = 0;
    writes = true;
    if constexpr (KG > 1) {
        constexpr int bit = 1 << SH;
        const bool up = lane & bit;
        if constexpr (NV % 2 == 0) {
            constexpr int h = NV / 2;
#pragma unroll
            for (int i = 0; i < h; ++i) {
                const A keep = up ? v[i + h] : v[i], give = up ? v[i] : v[i + h];
                v[i] = keep + __shfl_xor(give, bit, 64);
            }
            base = lane_reduce<A, h, KG / 2, SH + 1>(v, lane, writes) + (up ? h : 0);
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] += __shfl_xor(v[i], bit, 64);
            base = lane_reduce<A, NV, KG / 2, SH + 1>(v, lane, writes);
            writes = writes && !up;
        }
    }
    return base;
}
constexpr int left_after(int nv, int kg) { return kg == 1 ? nv : left_after(nv % 2 == 0 ? nv / 2 : nv, kg / 2); }
constexpr int log2i(int x) { return x <= 1 ? 0 : 1 + log2i(x / 2); }

// rows across lanes, and the waves per SIMD that the registers of the sums leave room for
constexpr int block_rows(int n) { return n % 16 == 0 ? 16 : 8; }
constexpr int block_waves(int n, int ct, int bytes) {
    const int sums = n / block_rows(n) * ct * bytes / 2;   // registers
    return sums >= 96 ? 2 : (sums >= 48 ? 3 : 4);
}

template <typename L, typename T, int N, bool DAG, bool WIL, int CT>
__global__ void __launch_bounds__(320) __attribute__((amdgpu_waves_per_eu(block_waves(N, CT, sizeof(typename acc_of<L>::type)))))
coarse_block_kernel(const L* __restrict__ links, const cpx<T>* __restrict__ in, cpx<T>* __restrict__ out,
                    const int* __restrict__ skip, int skip_stride, int Lx, int Ly, int Ls, int nsites, int ncol,
                    int tpb, typename acc_of<L>::type cdiag, typename acc_of<L>::type mwrap,
                    const cpx<T>* __restrict__ eb, T ealpha, T ebeta, double* __restrict__ norm, size_t norm_stride) {
    using A = typename acc_of<L>::type;
    constexpr int H = N / 2;
    constexpr int RI = block_rows(N);
    constexpr int KG = 64 / RI;                                          // inner indices across lanes
    constexpr int RT = N / RI;
    constexpr int KS = N / KG;
    static_assert(N % RI == 0 && N % KG == 0, "rows and inner indices fill the lanes");
    constexpr int KC = KS * RT <= 9 ? KS : (RT >= 4 ? 2 : (RT == 3 ? 3 : 4));   // inner steps in flight
    constexpr int NV = RT * CT * 2;
    constexpr int OUT = N * CT;                                          // outputs of a tile
    constexpr int PT = (OUT + 319) / 320;                                // outputs per thread
    __shared__ __attribute__((aligned(16))) cpx<A> sm[5][OUT];           // staged vectors, then the wave's part
    const int lane = threadIdx.x & 63;
    const int d = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int site = (int)xcd_block_dir<DAG>(blockIdx.x, gridDim.x);
    const int x = site % Lx, y = site / Lx;
    int nb = site;
    if (d == 1) nb = y * Lx + ((x + 1 == Lx) ? 0 : x + 1);
    else if (d == 2) nb = y * Lx + ((x == 0) ? Lx - 1 : x - 1);
    else if (d == 3) nb = ((y + 1 == Ly) ? 0 : y + 1) * Lx + x;
    else if (d == 4) nb = ((y == 0) ? Ly - 1 : y - 1) * Lx + x;
    const bool bwd = d == 2 || d == 4;
    // forward: element (i, k) at k N + i, rows on consecutive lanes; backward: conj of the
    // neighbour's (k, i), at i N + k, inner indices on consecutive lanes
    const int li = bwd ? lane / KG : lane % RI, kq = bwd ? lane % KG : lane / RI;
    const L* lk = links + ((size_t)(bwd ? nb : site) * 5 + (bwd ? d - 1 : d)) * N * N;
    // (a 32-bit byte offset per lane from bases that are the same for the whole wave)
    unsigned e0 = (unsigned)(bwd ? li * N + kq : kq * N + li) * (unsigned)sizeof(L);
    const int se_rt = bwd ? RI * N : RI, se_ks = bwd ? KG : KG * N;
    const A conj_sign = bwd ? A(-1) : A(1);
    L raw[KC][RT];   // the next KC inner steps: a step's registers are loaded again as soon as it is used
    auto load_step = [&](int ks) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const char* base = reinterpret_cast<const char*>(lk + (rt * se_rt + ks * se_ks));
            raw[ks % KC][rt] = *reinterpret_cast<const L*>(base + e0);
        }
    };
    const int C = Ls * ncol;
    const int ntile = (C + CT - 1) / CT;
    const int t_lo = (int)blockIdx.y * tpb, t_hi = min(ntile, t_lo + tpb);
    for (int t = t_lo; t < t_hi; ++t) {
        const int cbase = t * CT;
        // the tile's live columns, a flag per lane, loaded before the links so that waiting for it
        // does not wait for them (the same for all five waves)
        const bool col = lane < CT && cbase + lane < C;
        int flag = 0;
        if (skip) flag = skip[(size_t)((col ? cbase + lane : cbase) / Ls) * skip_stride];
#pragma unroll
        for (int ks = 0; ks < KC; ++ks) load_step(ks);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned alive = (unsigned)__ballot(col && flag == 0);
        if (alive == 0) continue;
        auto live = [&](int c) { return ((alive >> (c - cbase)) & 1u) != 0; };
        // this wave's neighbour vectors: columns past the end or stopped are zero; sigma_3 on
        // the vector for the adjoint and for the sigma_3-adjoint links
#pragma unroll
        for (int p = 0; p < (OUT + 63) / 64; ++p) {
            const int e = p * 64 + lane;
            if (OUT % 64 == 0 || e < OUT) {
                const int k = e % N, c = e / N;
                cpx<A> v = {A(0), A(0)};
                if (live(cbase + c)) {
                    const cpx<T> g = in[((size_t)(cbase + c) * nsites + nb) * N + k];
                    v = {(A)g.re, (A)g.im};
                    if (k >= H && DAG != bwd) v = {-v.re, -v.im};
                }
                sm[d][k * CT + c] = v;
            }
        }
        // the site-local terms of this thread's outputs, loaded while the products run
        cpx<T> lc[PT], lh[PT], le[PT];
        bool wr[PT];
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int o = (int)threadIdx.x + p * 320;
            wr[p] = o < OUT && live(cbase + o / N);
            lc[p] = lh[p] = le[p] = cpx<T>{T(0), T(0)};
            if (wr[p]) {
                const int i = o % N, c = cbase + o / N;
                lc[p] = in[((size_t)c * nsites + site) * N + i];
                if (!WIL) {
                    const int s = c % Ls;
                    const int so = (DAG != (i >= H)) ? (s + 1 == Ls ? 0 : s + 1) : (s == 0 ? Ls - 1 : s - 1);
                    lh[p] = in[((size_t)(c - s + so) * nsites + site) * N + i];
                }
                if (eb) le[p] = eb[((size_t)c * nsites + site) * N + i];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        A v[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = A(0);
        int l0 = kq * CT;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const cpx<A>* pv = &sm[d][ks * KG * CT + l0];
            cpx<A> w[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) w[c] = pv[c];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                cpx<A> l = load_link(raw[ks % KC], rt);
                l.im *= conj_sign;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    A& re = v[(rt * CT + c) * 2];
                    A& im = v[(rt * CT + c) * 2 + 1];
                    re = fma(l.re, w[c].re, re);
                    im = fma(l.re, w[c].im, im);
                    re = fma(-l.im, w[c].im, re);
                    im = fma(l.im, w[c].re, im);
                }
            }
            // this step's sums are formed before the loads of later steps (empty asm statements take
            // the sums and give back the addresses): left to itself the compiler puts most of the
            // sums off behind the last load and spills
#pragma unroll
            for (int q = 0; q < NV; ++q) asm volatile("" : "+v"(v[q]));
            asm volatile("" : "+v"(e0), "+v"(l0));
            if (ks + KC < KS) load_step(ks + KC);
        }
        // sum over the kq lanes, then this wave's part over its staged vectors (its own LDS
        // operations complete in order)
        auto leave_part = [&](auto shc) {
            bool writes;
            constexpr int LEFT = left_after(NV, KG);
            const int base = lane_reduce<A, NV, KG, decltype(shc)::value>(v, lane, writes);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (writes) {
                A* pt = reinterpret_cast<A*>(&sm[d][0]);
#pragma unroll
                for (int q = 0; q < LEFT; ++q) {
                    const int e = base + q, ri = e & 1, c = (e >> 1) % CT, rt = (e >> 1) / CT;
                    pt[(c * N + rt * RI + li) * 2 + ri] = v[q];
                }
            }
        };
        if (bwd) leave_part(std::integral_constant<int, 0>{});
        else leave_part(std::integral_constant<int, log2i(RI)>{});
        __syncthreads();
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int o = (int)threadIdx.x + p * 320;
            if (!wr[p]) continue;
            const int i = o % N, c = cbase + o / N;
            const bool minus = i >= H;
            cpx<A> f = sm[0][o] + sm[1][o] + sm[3][o], g = sm[2][o] + sm[4][o];
            // row signs: sigma_3 of the adjoint on all, of the sigma_3-adjoint links on the backward hops
            if (minus && DAG) f = {-f.re, -f.im};
            if (minus && !DAG) g = {-g.re, -g.im};
            cpx<A> r = f + g;
            r.re += cdiag * (A)lc[p].re;
            r.im += cdiag * (A)lc[p].im;
            if (!WIL) {
                const int s = c % Ls;
                const A h = ((DAG != minus) ? s + 1 == Ls : s == 0) ? mwrap : A(1);
                r.re += h * (A)lh[p].re;
                r.im += h * (A)lh[p].im;
            }
            cpx<T> w = {(T)r.re, (T)r.im};
            if (eb) w = {ealpha * w.re + ebeta * le[p].re, ealpha * w.im + ebeta * le[p].im};
            out[((size_t)c * nsites + site) * N + i] = w;
            // (a thread reads only its own outputs' parts: their place takes |out|^2)
            if (norm) *reinterpret_cast<double*>(&sm[0][o]) = (double)w.re * w.re + (double)w.im * w.im;
        }
        if (norm) {   // (uniform) one partial per (column, site)
            __syncthreads();
            const int c = cbase + (int)threadIdx.x;
            if ((int)threadIdx.x < CT && live(c)) {
                double sum = 0.0;
#pragma unroll 8
                for (int i = 0; i < N; ++i) sum += *reinterpret_cast<const double*>(&sm[0][threadIdx.x * N + i]);
                norm[(size_t)(c / Ls) * norm_stride + (size_t)(c % Ls) * nsites + site] = sum;
            }
        }
        if (t + 1 < t_hi) __syncthreads();   // the next tile stages over the parts
    }
}

namespace {

template <typename L, typename T, int N>
hipError_t launch_n(const void* links, const cpx<T>* in, cpx<T>* out, const CoarseGeom& g, int ncol,
                    double m, double M5, bool dagger, bool wil, double wmass, const int* skip, int sks, hipStream_t st,
                    const Epi<T>& epi) {
    using A = typename acc_of<L>::type;
    const int nsites = g.Lx * g.Ly;
    const L* lk = reinterpret_cast<const L*>(links);
    const A cd = wil ? (A)wmass : (A)(M5 + 1.0);
    const A mw = (A)(-m);
    const T ea = (T)epi.alpha, ebt = (T)epi.beta;
    // (the 2-d operator is applied with FP64 links alone: setup and diagnostics)
    auto with_op = [&](auto go) {
        if constexpr (std::is_same_v<L, cpx<double>>) {
            if (wil) return dagger ? go(std::true_type{}, std::true_type{}) : go(std::false_type{}, std::true_type{});
        } else if (wil) {
            return hipErrorInvalidValue;
        }
        return dagger ? go(std::true_type{}, std::false_type{}) : go(std::false_type{}, std::false_type{});
    };
    if constexpr (N >= 16) {
        // column tiles of 2, 4 or 8, all of a site's in one workgroup (its later tiles then find
        // the links in L2) unless the sites alone would leave compute units without one
        const int C = g.Ls * ncol;
        const int ct = C <= 2 ? 2 : (C <= 4 ? 4 : 8);
        const int ntile = (C + ct - 1) / ct;
        const int gy0 = std::min(ntile, std::max(1, 1024 / nsites));
        const int tpb = (ntile + gy0 - 1) / gy0;
        const dim3 grid(nsites, (ntile + tpb - 1) / tpb), block(320);
        auto with_ct = [&](auto ctc) {
            return with_op([&](auto dagc, auto wilc) {
                hipLaunchKernelGGL((coarse_block_kernel<L, T, N, decltype(dagc)::value, decltype(wilc)::value,
                                                        decltype(ctc)::value>),
                                   grid, block, 0, st, lk, in, out, skip, sks, g.Lx, g.Ly, g.Ls, nsites, ncol, tpb, cd, mw,
                                   epi.b, ea, ebt, epi.norm, epi.norm_stride);
                return hipGetLastError();
            });
        };
        if (ct == 2) return with_ct(std::integral_constant<int, 2>{});
        if (ct == 4) return with_ct(std::integral_constant<int, 4>{});
        return with_ct(std::integral_constant<int, 8>{});
    } else {
        size_t per_wave_bytes = (size_t)coarse_lds_per_wave(N, g.Ls) * sizeof(cpx<A>);
        int wpb = 4;
        while (wpb > 1 && per_wave_bytes * wpb > 64 * 1024) wpb >>= 1;
        if (per_wave_bytes * wpb > 160 * 1024) return hipErrorInvalidValue;
        const dim3 grid((nsites + wpb - 1) / wpb, ncol), block(64 * wpb);
        return with_op([&](auto dagc, auto wilc) {
            hipLaunchKernelGGL((coarse_kernel<L, T, N, decltype(dagc)::value, decltype(wilc)::value>), grid, block,
                               per_wave_bytes * wpb, st, lk, in, out, skip, sks, g.Lx, g.Ly, g.Ls, nsites, cd, mw, epi.b,
                               ea, ebt);
            return hipGetLastError();
        });
    }
}

// (16-bit links of a multiple of 16 components go to the matrix cores: coarse_mfma_supported)
template <typename L, typename T, int N, typename... Args>
hipError_t launch_valu(const Args&... args) {
    if constexpr (sizeof(L) == 4 && N % 16 == 0) return hipErrorInvalidValue;
    else return launch_n<L, T, N>(args...);
}

template <typename L, typename T>
hipError_t launch_l(const void* links, const cpx<T>* in, cpx<T>* out, const CoarseGeom& g, int ncol,
                    double m, double M5, bool dagger, bool wil, double wmass, const int* skip, int sks, hipStream_t st,
                    const Epi<T>& epi) {
    switch (g.n) {
        case 4:  return launch_valu<L, T, 4>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        case 8:  return launch_valu<L, T, 8>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        case 12: return launch_valu<L, T, 12>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        case 16: return launch_valu<L, T, 16>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        case 24: return launch_valu<L, T, 24>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        case 32: return launch_valu<L, T, 32>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        case 48: return launch_valu<L, T, 48>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        case 64: return launch_valu<L, T, 64>(links, in, out, g, ncol, m, M5, dagger, wil, wmass, skip, sks, st, epi);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool coarse_norm_supported(int n, int link_prec) { return n >= 16 && !coarse_mfma_supported(n, link_prec); }

template <typename T>
hipError_t coarse_apply(const void* links, int link_prec, const cpx<T>* in, cpx<T>* out,
                        const CoarseGeom& g, int ncol, double m, double M5, bool dagger,
                        bool wilson_mode, double wilson_mass, const int* skip, int sks, hipStream_t st,
                        const Epi<T>& epi) {
    if (g.Ls < 1 || g.Ls > kMaxCoarseLs) return hipErrorInvalidValue;
    if (epi.norm && (wilson_mode || !coarse_norm_supported(g.n, link_prec))) return hipErrorInvalidValue;
    if (!wilson_mode && coarse_mfma_supported(g.n, link_prec))
        return coarse_apply_mfma<T>(links, link_prec, in, out, g, ncol, m, M5, dagger, skip, sks, st, epi);
    switch (link_prec) {
        case P_F64: return launch_l<cpx<double>, T>(links, in, out, g, ncol, m, M5, dagger, wilson_mode, wilson_mass, skip, sks, st, epi);
        case P_F32: return launch_l<cpx<float>, T>(links, in, out, g, ncol, m, M5, dagger, wilson_mode, wilson_mass, skip, sks, st, epi);
        case P_BF16: return launch_l<cbf16, T>(links, in, out, g, ncol, m, M5, dagger, wilson_mode, wilson_mass, skip, sks, st, epi);
        case P_F16: return launch_l<cf16, T>(links, in, out, g, ncol, m, M5, dagger, wilson_mode, wilson_mass, skip, sks, st, epi);
        default: return hipErrorInvalidValue;
    }
}

template hipError_t coarse_apply<float>(const void*, int, const cpx<float>*, cpx<float>*, const CoarseGeom&, int, double, double, bool, bool, double, const int*, int, hipStream_t, const Epi<float>&);
template hipError_t coarse_apply<double>(const void*, int, const cpx<double>*, cpx<double>*, const CoarseGeom&, int, double, double, bool, bool, double, const int*, int, hipStream_t, const Epi<double>&);

}  // namespace dwf
