// RBF interpolation (Sec. 2): the Gaussian smoothing sums that form the
// matrix-vector product of the interpolation system, and the vector kernels
// of its GMRES iteration.
//
// Gaussian sums over the neighbour list of the tree: for a target in leaf c,
// every source in the 27 leaves c + d (periodic: wrapped, with the image
// shift), omega_i = (2 pi sigma^2)^(-3/2) sum_j gamma_j exp(-r_ij^2 / (2 sigma^2)).
// One target per lane; the source records (position relative to the leaf centre,
// strength gamma in the a-fields) are read at wave-uniform addresses (scalar
// loads).  Leaves go to waves as in leaf_sums.h: split over the waves of a
// workgroup on small trees (32^3, FP64: 64 us a product, 194 with one wave per leaf and
// the library's exponential).  Vectors are in the sorted particle
// order, [3][n] FP64.
#include "leaf_sums.h"

namespace vmfmm {

namespace {

// One source against the lane's target: scaled coordinates, c = sqrt(log2(e)
// / (2 sigma^2)), so that exp(-r^2 / (2 sigma^2)) = 2^-(|c r|^2) and c r =
// c t - c s takes one FMA per axis.
__device__ __forceinline__ float exp2_minus(float q, uint32_t) { return __builtin_amdgcn_exp2f(-q); }

// FP64: 2^-q = 2^-(k / 64) 2^-f, k = rint(64 q), |f| <= 1/128: 64 powers in LDS and
// the Taylor series of degree 5 (truncation 3.5e-17), 17 instructions against the
// library's 40.
constexpr double kLn2 = 0.69314718055994530942;
__device__ __forceinline__ double exp2_minus(double q, uint32_t tab) {
    q = q > 1100.0 ? 1100.0 : q;   // 0 (2^-1100 underflows); NaN stays
    const double kf = rint(q * 64.0);
    const double f = fma(kf, -0.015625, q);   // exact
    const int k = int(kf);
    typedef const __attribute__((address_space(3))) double *P;
    const double p64 = *(P)(tab + 8u * uint32_t(k & 63));
    constexpr double c1 = -kLn2, c2 = kLn2 * kLn2 / 2, c3 = -kLn2 * kLn2 * kLn2 / 6,
                     c4 = kLn2 * kLn2 * kLn2 * kLn2 / 24, c5 = -kLn2 * kLn2 * kLn2 * kLn2 * kLn2 / 120;
    double p = fma(c5, f, c4);
    p = fma(p, f, c3);
    p = fma(p, f, c2);
    p = fma(p, f, c1);
    p = p * f;                     // 2^-f - 1
    return ldexp(fma(p64, p, p64), -(k >> 6));
}

// Sums over the neighbour leaves (leaf_sums.h).  T: arithmetic of the pair (double:
// FP64 form; float: mixed form, FP32 differences, exponential and sums over a
// source leaf's share, added into FP64 sums).
template <typename T, typename P>
struct GaussPol {
    using Rec = P;
    using Real = T;
    struct Acc {
        double s[3];
    };
    T c, mc;
    double norm;
    uint32_t tab;
    __device__ __forceinline__ T scaled(T x) const { return c * x; }
    static __device__ __forceinline__ void clear(Acc &A) { A.s[0] = A.s[1] = A.s[2] = 0.0; }
    __device__ __forceinline__ void pair(const P &src, T cx, T cy, T cz, T part[3]) const {
        const T rx = fma(T(src.dx), mc, cx), ry = fma(T(src.dy), mc, cy), rz = fma(T(src.dz), mc, cz);
        const T e = exp2_minus(rx * rx + ry * ry + rz * rz, tab);
        part[0] = fma(T(src.ax), e, part[0]);
        part[1] = fma(T(src.ay), e, part[1]);
        part[2] = fma(T(src.az), e, part[2]);
    }
    __device__ __forceinline__ void uniform(const P *__restrict__ parts, int js, int je, T tx, T ty, T tz,
                                            Acc &A) const {
        T part[3] = {T(0), T(0), T(0)};
        int j = js;
        for (; j + 4 <= je; j += 4) {
            const P s0 = parts[j], s1 = parts[j + 1], s2 = parts[j + 2], s3 = parts[j + 3];
            pair(s0, tx, ty, tz, part);
            pair(s1, tx, ty, tz, part);
            pair(s2, tx, ty, tz, part);
            pair(s3, tx, ty, tz, part);
        }
        for (; j < je; ++j) pair(parts[j], tx, ty, tz, part);
        for (int q = 0; q < 3; ++q) A.s[q] += double(part[q]);
    }
    __device__ __forceinline__ void grouped(const P *__restrict__ parts, int js, int je, int ng, T tx, T ty, T tz,
                                            Acc &A) const {
        T part[3] = {T(0), T(0), T(0)};
#pragma unroll 1
        for (int j = js; j < je; j += ng) pair(parts[j], tx, ty, tz, part);
        for (int q = 0; q < 3; ++q) A.s[q] += double(part[q]);
    }
    template <int K>
    __device__ __forceinline__ double value(const Acc &A) const {
        if constexpr (K < 3) return norm * A.s[K];
        else return 0.0;
    }
};

template <typename T, typename P, bool SPLIT>
// FP32: 8 waves a SIMD (64 registers) hide the scalar loads.  A tree that fills the
// chip takes one wave per workgroup: no workgroup of 8 then waits for its fullest
// leaf (32768 leaves of 64: 1.04 ms a product; 8 waves a workgroup, 7 a SIMD 1.07).
__global__ void __launch_bounds__(SPLIT ? kP2PThreads : 64)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 8 : 4, 8))) k_gauss(P2PArgs a, const P *__restrict__ parts) {
    __shared__ double red[SPLIT ? kRedDoubles : 1];
    __shared__ double pow2[sizeof(T) == 8 ? 64 : 1];
    GaussPol<T, P> pol;
    if constexpr (sizeof(T) == 8) {
        if (threadIdx.x < 64) pow2[threadIdx.x] = exp2(-double(threadIdx.x) / 64.0);
        __syncthreads();
    }
    const double c64 = sqrt(0.5 * 1.4426950408889634074) / a.sigma;
    const double s2pi = 2.0 * 3.14159265358979323846 * a.sigma * a.sigma;
    pol.c = T(c64);
    pol.mc = -pol.c;
    pol.norm = 1.0 / (s2pi * sqrt(s2pi));
    pol.tab = uint32_t(uintptr_t((const __attribute__((address_space(3))) double *)pow2));
    p2p_leaves<GaussPol<T, P>, SPLIT>(a, parts, pol, red);
}

// v <- alpha v0 and parts[i].a = v[:][i] (sorted order): the next product's strengths
template <typename P, typename S>
__global__ void __launch_bounds__(256) k_scale_pack(int n, const double *v0, double *v, double a0, double a1,
                                                    double a2, P *__restrict__ parts) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const size_t m = size_t(n);
    const double x = a0 * v0[i], y = a1 * v0[m + i], z = a2 * v0[2 * m + i];
    v[i] = x;
    v[m + i] = y;
    v[2 * m + i] = z;
    parts[i].ax = S(x);
    parts[i].ay = S(y);
    parts[i].az = S(z);
}

// dst[c][i] = src[c][perm[i]] (caller order -> sorted order)
__global__ void __launch_bounds__(256) k_gather3(int n, const int32_t *__restrict__ perm,
                                                 const double *__restrict__ src, double *__restrict__ dst) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int j = perm[i];
    if (j < 0 || j >= n) return;   // never for a valid permutation
    for (int c = 0; c < 3; ++c) dst[size_t(c) * n + i] = src[size_t(c) * n + j];
}

// dst[c][perm[i]] = scale * src[c][i] (sorted order -> caller order)
__global__ void __launch_bounds__(256) k_scatter3(int n, const int32_t *__restrict__ perm,
                                                  const double *__restrict__ src, double scale,
                                                  double *__restrict__ dst) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int j = perm[i];
    if (j < 0 || j >= n) return;
    for (int c = 0; c < 3; ++c) dst[size_t(c) * n + j] = scale * src[size_t(c) * n + i];
}

// Vectors and dot products of one Arnoldi step, bounded by the passes over the
// basis: workgroup (x, c) takes component c of a grid-stride share of the
// particles.  Row r = 3 j + c of a dot product holds its workgroups' partial sums
// at partial[r kRbfDotBlocks + x]; the consumer adds them in a fixed order.
template <int K>
__device__ __forceinline__ void block_sums(const double (&s)[K], int k, int c, double *__restrict__ partial) {
    __shared__ double red[K][4];
    const int tid = threadIdx.x;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (q >= k) break;
        double x = s[q];
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
        if ((tid & 63) == 0) red[q][tid >> 6] = x;
    }
    __syncthreads();
    if (tid < k)
        partial[size_t(3 * tid + c) * kRbfDotBlocks + blockIdx.x] =
            (red[tid][0] + red[tid][1]) + (red[tid][2] + red[tid][3]);
}

// row r of a partial, all lanes of the wave
__device__ __forceinline__ double row_sum(const double *__restrict__ partial, int r, int nb) {
    double s = 0.0;
    for (int b = threadIdx.x & 63; b < nb; b += 64) s += partial[size_t(r) * kRbfDotBlocks + b];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    return s;
}

// Gram-Schmidt: h = the dot products in `pin` (to out, row order), w <- w - sum_j
// h_j v_j where the component's bit of `active` is set (UPD), and the dot
// products of the new w with v_j, j < k (K > 0: K >= k, the basis read once and
// held), or its square (K = 0), to pout.  The update and the dot products that
// follow it share a pass, and each workgroup adds the partial sums itself, so a
// step is 4 launches with one wait for the host at its end; apart and with the
// host in between it was 11 launches and 3 waits (32^3, 4 vectors: 245 us from
// product to product, now 54).
template <int K, bool UPD>
__global__ void __launch_bounds__(256) k_arnoldi(int n, double *__restrict__ w, const double *__restrict__ V,
                                                 int64_t ldv, int k, int active, const double *__restrict__ pin,
                                                 double *__restrict__ out, double *__restrict__ pout) {
    __shared__ double h[kRbfMaxVecs];
    const int tid = threadIdx.x, c = blockIdx.y, nb = gridDim.x;
    if constexpr (UPD) {
        for (int j = tid >> 6; j < k; j += 4) {
            const double x = row_sum(pin, 3 * j + c, nb);
            if ((tid & 63) == 0) {
                h[j] = active >> c & 1 ? -x : 0.0;
                if (blockIdx.x == 0) out[3 * j + c] = x;
            }
        }
        __syncthreads();
    }
    w += size_t(c) * size_t(n);
    V += size_t(c) * size_t(n);
    constexpr int KS = K > 0 ? K : 1;
    double s[KS] = {};
    for (int64_t i = int64_t(blockIdx.x) * 256 + tid; i < n; i += int64_t(nb) * 256) {
        double x = w[i];
        if constexpr (K > 0) {
            double v[K];
#pragma unroll
            for (int q = 0; q < K; ++q) v[q] = q < k ? V[q * ldv + i] : 0.0;
            if constexpr (UPD) {
#pragma unroll
                for (int q = 0; q < K; ++q)
                    if (q < k) x = fma(h[q], v[q], x);
                w[i] = x;
            }
#pragma unroll
            for (int q = 0; q < K; ++q) s[q] = fma(x, v[q], s[q]);
        } else {
            for (int j = 0; j < k; ++j) x = fma(h[j], V[j * ldv + i], x);
            w[i] = x;
            s[0] = fma(x, x, s[0]);
        }
    }
    block_sums(s, K > 0 ? k : 1, c, pout);
}

// r <- b - r and its square
__global__ void __launch_bounds__(256) k_residual(int n, const double *__restrict__ b, double *__restrict__ r,
                                                  double *__restrict__ pout) {
    const int c = blockIdx.y;
    b += size_t(c) * size_t(n);
    r += size_t(c) * size_t(n);
    double s[1] = {0.0};
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        const double x = b[i] - r[i];
        r[i] = x;
        s[0] = fma(x, x, s[0]);
    }
    block_sums(s, 1, c, pout);
}

// host[0 .. nh) = h, then the three squares of `partial`: what the host reads of a step
__global__ void __launch_bounds__(256) k_arnoldi_read(int nb, const double *__restrict__ partial, int nh,
                                                      const double *__restrict__ h, double *__restrict__ host) {
    const int tid = threadIdx.x, c = tid >> 6;
    for (int i = tid; i < nh; i += 256) host[i] = h[i];
    if (c >= 3) return;
    const double s = row_sum(partial, c, nb);
    if ((tid & 63) == 0) host[nh + c] = s;
}

// w[c][i] = alpha_c w[c][i] + sum_{j < k} c_{j,c} v_j[c][i]
__global__ void __launch_bounds__(256) k_multiaxpy(int n, double *__restrict__ w, const double *__restrict__ V,
                                                   int64_t ldv, int k, RbfCoefs cf) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const size_t m = size_t(n);
    for (int c = 0; c < 3; ++c) {
        double s = cf.alpha[c] * w[c * m + i];
        for (int j = 0; j < k; ++j) s = fma(cf.c[3 * j + c], V[j * ldv + c * m + i], s);
        w[c * m + i] = s;
    }
}

// Cell centres of the ng^3 lattice on the box: site k = (ix ng + iy) ng + iz
// at lo + (i + 1/2) h, written as [3][ng^3].
__global__ void __launch_bounds__(256) k_lattice_sites(int ng, double lo0, double lo1, double lo2, double h,
                                                       double *__restrict__ out) {
    const int n = ng * ng * ng;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const int ix = k / (ng * ng), iy = (k / ng) % ng, iz = k % ng;
    const size_t m = size_t(n);
    out[k] = lo0 + (double(ix) + 0.5) * h;
    out[m + k] = lo1 + (double(iy) + 0.5) * h;
    out[2 * m + k] = lo2 + (double(iz) + 0.5) * h;
}

unsigned blocks256(int n) { return unsigned((n + 255) / 256); }

}  // namespace

hipError_t launch_gauss(hipStream_t s, const GaussArgs &g, const void *parts, int mixed) {
    P2PArgs a{};
    a.n = g.n;
    a.nleaf = g.nleaf;
    a.level = g.level;
    a.periodic = g.periodic;
    a.w = g.w;
    a.sigma = g.sigma;
    a.start = g.start;
    a.tstart = g.tstart;
    a.tparts = g.tparts;
    a.near = g.out;   // rows 0 .. 2
    P2PShape p = p2p_shape(a, compute_units() * 4, 0);
    if (!p.split) p.grid.x = unsigned(a.nleaf);
    const dim3 wg(p.split ? kP2PThreads : 64);
    if (mixed) {
        const auto k = p.split ? k_gauss<float, Part32, true> : k_gauss<float, Part32, false>;
        hipLaunchKernelGGL(k, p.grid, wg, 0, s, a, (const Part32 *)parts);
    } else {
        const auto k = p.split ? k_gauss<double, Part64, true> : k_gauss<double, Part64, false>;
        hipLaunchKernelGGL(k, p.grid, wg, 0, s, a, (const Part64 *)parts);
    }
    return hipGetLastError();
}

hipError_t launch_scale_pack(hipStream_t s, int n, const double *v0, double *v, const double alpha[3], void *parts,
                             int mixed) {
    if (mixed)
        hipLaunchKernelGGL((k_scale_pack<Part32, float>), dim3(blocks256(n)), dim3(256), 0, s, n, v0, v, alpha[0],
                           alpha[1], alpha[2], (Part32 *)parts);
    else
        hipLaunchKernelGGL((k_scale_pack<Part64, double>), dim3(blocks256(n)), dim3(256), 0, s, n, v0, v, alpha[0],
                           alpha[1], alpha[2], (Part64 *)parts);
    return hipGetLastError();
}

hipError_t launch_lattice_sites(hipStream_t s, int ng, const double lo[3], double h, double *out) {
    const int n = ng * ng * ng;
    hipLaunchKernelGGL(k_lattice_sites, dim3(blocks256(n)), dim3(256), 0, s, ng, lo[0], lo[1], lo[2], h, out);
    return hipGetLastError();
}

hipError_t launch_gather3(hipStream_t s, int n, const int32_t *perm, const double *src, double *dst) {
    hipLaunchKernelGGL(k_gather3, dim3(blocks256(n)), dim3(256), 0, s, n, perm, src, dst);
    return hipGetLastError();
}

hipError_t launch_scatter3(hipStream_t s, int n, const int32_t *perm, const double *src, double scale, double *dst) {
    hipLaunchKernelGGL(k_scatter3, dim3(blocks256(n)), dim3(256), 0, s, n, perm, src, scale, dst);
    return hipGetLastError();
}

static dim3 arnoldi_grid(int n) { return dim3(std::min(unsigned(kRbfDotBlocks), blocks256(n)), 3); }

template <bool UPD>
static hipError_t arnoldi(hipStream_t s, int n, double *w, const double *V, int64_t ldv, int k, int active,
                          const double *pin, double *out, double *pout) {
    const auto f = k <= 4 ? k_arnoldi<4, UPD> : k <= 8 ? k_arnoldi<8, UPD> : k <= 12 ? k_arnoldi<12, UPD>
                                              : k <= 16 ? k_arnoldi<16, UPD> : k_arnoldi<kRbfMaxDots, UPD>;
    hipLaunchKernelGGL(f, arnoldi_grid(n), dim3(256), 0, s, n, w, V, ldv, k, active, pin, out, pout);
    return hipGetLastError();
}

hipError_t launch_orthogonalize(hipStream_t s, int n, double *w, const double *V, int64_t ldv, int k, int active,
                                double *partial, double *h, double *host) {
    if (k < 1 || k > kRbfMaxDots) return hipErrorInvalidValue;
    double *p0 = partial, *p1 = partial + size_t(3) * kRbfMaxVecs * kRbfDotBlocks;
    hipError_t e = arnoldi<false>(s, n, w, V, ldv, k, active, nullptr, nullptr, p0);
    if (e == hipSuccess) e = arnoldi<true>(s, n, w, V, ldv, k, active, p0, h, p1);
    if (e != hipSuccess) return e;
    const dim3 g = arnoldi_grid(n);
    hipLaunchKernelGGL((k_arnoldi<0, true>), g, dim3(256), 0, s, n, w, V, ldv, k, active, p1, h + 3 * k, p0);
    hipLaunchKernelGGL(k_arnoldi_read, dim3(1), dim3(256), 0, s, int(g.x), p0, 6 * k, h, host);
    return hipGetLastError();
}

hipError_t launch_residual(hipStream_t s, int n, const double *b, double *r, double *partial, double *host) {
    const dim3 g = arnoldi_grid(n);
    hipLaunchKernelGGL(k_residual, g, dim3(256), 0, s, n, b, r, partial);
    hipLaunchKernelGGL(k_arnoldi_read, dim3(1), dim3(256), 0, s, int(g.x), partial, 0, (const double *)nullptr, host);
    return hipGetLastError();
}

hipError_t launch_multiaxpy(hipStream_t s, int n, double *w, const double *V, int64_t ldv, int k,
                            const RbfCoefs &c) {
    hipLaunchKernelGGL(k_multiaxpy, dim3(blocks256(n)), dim3(256), 0, s, n, w, V, ldv, k, c);
    return hipGetLastError();
}

}  // namespace vmfmm
