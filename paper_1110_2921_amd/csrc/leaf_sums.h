// Sums over the neighbour leaves of a uniform tree (near field, Gaussian sums): how
// a launch deals leaves, targets and sources to workgroups, waves and lanes.  The
// pair arithmetic comes as a policy POL: Rec and Real (record and arithmetic
// types), scaled() (the policy's unit of length), Acc with clear(), uniform() (sources js .. je - 1 at wave-uniform
// addresses against the lane's target), grouped() (every ng-th source from js on)
// and value<K>() (row K of the sums, FP64).
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "kernels.h"

namespace vmfmm {
namespace {

constexpr double kInv4Pi = 0.079577471545947667884441881686257181;

__device__ __forceinline__ int demorton(int k, int d, int level) {
    int c = 0;
    for (int b = 0; b < level; ++b) c |= ((k >> (3 * b + d)) & 1) << b;
    return c;
}

__device__ __forceinline__ int morton(int cx, int cy, int cz, int level) {
    int k = 0;
    for (int b = 0; b < level; ++b)
        k |= (((cx >> b) & 1) << (3 * b)) | (((cy >> b) & 1) << (3 * b + 1)) | (((cz >> b) & 1) << (3 * b + 2));
    return k;
}

struct LeafGeom {
    int cx, cy, cz, side;
};

// neighbour nb of the target leaf: source range and the offset d (source - target cell)
__device__ __forceinline__ bool neighbour(const P2PArgs &a, const LeafGeom &L, int nb, int &js, int &je, int &dx,
                                          int &dy, int &dz) {
    dx = nb % 3 - 1;
    dy = (nb / 3) % 3 - 1;
    dz = nb / 9 - 1;
    int nx = L.cx + dx, ny = L.cy + dy, nz = L.cz + dz;
    if (a.periodic) {
        nx = (nx + L.side) % L.side;
        ny = (ny + L.side) % L.side;
        nz = (nz + L.side) % L.side;
    } else if (nx < 0 || ny < 0 || nz < 0 || nx >= L.side || ny >= L.side || nz >= L.side) {
        return false;
    }
    const int nk = morton(nx, ny, nz, a.level);
    js = a.start[nk];
    je = a.start[nk + 1];
    return true;
}

// Workgroups of 8 waves (the pair table in LDS is shared), one target per lane,
// sources at wave-uniform addresses (scalar loads).  Two ways to deal out the
// work:
//   SPLIT   a workgroup takes one leaf at a time: the sources of its 27
//           neighbour leaves, concatenated, go to the waves in equal contiguous
//           shares, every wave holds the same targets, and the waves' sums are
//           added through LDS in wave order.  A tree of few leaves needs this:
//           with one wave per leaf, 64 leaves ran 64 waves on 1024 SIMDs, each
//           through 1728 sources in turn (16^3 FP64: 602 us; split 30 us).
//           Trees of fewer leaves than the chip holds workgroups also deal a
//           leaf's target blocks over gridDim.y and its sources over gridDim.z
//           (partial near fields, added by L2P).
//   !SPLIT  a wave per leaf, without the reduction, from kP2PSplitLeaves on, where
//           the leaves fill the chip many times over (128^3, one evaluation:
//           FP64 13.7 against 14.5 ms split, a mixed Heun step 14.6 against 15.9).
// Workgroups go to the 8 XCDs round-robin, so workgroup b takes leaves of the
// (b mod 8)-th eighth of the Morton order, whose neighbour leaves that XCD's L2
// then shares.
constexpr int kP2PWaves = 8;
constexpr int kP2PThreads = 64 * kP2PWaves;
constexpr int kNearRows = 15;     // u, gradient sums, strength sums
constexpr int kRedRows = 3;       // values per reduction round
constexpr int kRedDoubles = kRedRows * kP2PThreads + kNearRows * 64;

// lane group size of a target piece of `rem` targets: 64 (a whole wave) or the
// lane groups' power of two; a remainder a little over a power of two is cut
// there, the rest is a piece of its own (34 targets: 32 + 2, 34 / 64 of a
// whole-wave pass instead of all of it)
__device__ __forceinline__ int piece_lanes(int rem) {
    if (rem > 48) return 64;
    int e = 1;
    while (e < rem) e <<= 1;
    return e > 8 && 4 * rem <= 3 * e ? e >> 1 : e;
}

template <int K>
using IC = std::integral_constant<int, K>;

template <class F, int... K>
__device__ __forceinline__ void for_rows(F &&f, std::integer_sequence<int, K...>) {
    (f(IC<K>{}), ...);
}

// Rows kRedRows R .. of the waves' sums sum(row), added through LDS in wave order;
// put(row, x) gets the lane's total in the threads below 64 kRedRows
template <int R, class F, class G>
__device__ __forceinline__ void wave_round(double *red, F sum, G put) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for_rows([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        red[(k * kP2PWaves + wave) * 64 + lane] = sum(IC<R * kRedRows + k>{});
    }, std::make_integer_sequence<int, kRedRows>{});
    __syncthreads();
    if (tid < 64 * kRedRows) {
        const int k = tid >> 6;
        double x = 0.0;
#pragma unroll
        for (int q = 0; q < kP2PWaves; ++q) x += red[(k * kP2PWaves + q) * 64 + lane];
        put(R * kRedRows + k, x);
    }
    __syncthreads();
}

// u, J and dalpha/dt of sorted target gi from its near sums f(row), with the
// far field where there is one, in caller order
template <class F>
__device__ __forceinline__ void finish(const P2PArgs &a, int gi, bool write, F f) {
    if (!write) return;
    const size_t n = size_t(a.n);
    const int oi = a.perm[gi];
    for (int b = 0; b < 3; ++b) a.u[b * n + oi] = f(b) * kInv4Pi + (a.have_far ? a.far[b * n + gi] : 0.0);
    if (!a.grad && !a.dalpha) return;
    double al[3] = {0.0, 0.0, 0.0};
    if (a.dalpha)
        for (int c = 0; c < 3; ++c) al[c] = a.alpha[c * n + oi];
    double da[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            // antisymmetric part eps_abc S_c of the near gradient J[r][c]
            const int k = 3 - r - c;
            const double anti = r == c ? 0.0 : ((c == (r + 1) % 3) ? f(12 + k) : -f(12 + k));
            double J = (f(3 + 3 * r + c) + anti) * kInv4Pi;
            if (a.have_far) J += a.far[(3 + 3 * r + c) * n + gi];
            if (a.grad) a.grad[(3 * r + c) * n + oi] = J;
            if (a.scheme == 0) da[c] += al[r] * J;      // classic: sum_a alpha_a J[a][b]
            else da[r] += J * al[c];                     // transpose: sum_c J[b][c] alpha_c
        }
    }
    if (a.dalpha)
        for (int b = 0; b < 3; ++b) a.dalpha[b * n + oi] = da[b];
}

// The sum over lane groups of E lanes (fixed butterfly), in every lane.  Where waves share
// a leaf it is taken of the waves' sums: of each wave's it kept the LDS busy with
// eight times the exchanges (50000 particles at level 4, P2P mixed 232 us, now 208, FP64
// 267 and 223; an evaluation of 2^19 in an adaptive tree 9.38 ms, now 9.20).
__device__ __forceinline__ double group_sum(double x, int E) {
    for (int off = E; off < 64; off <<= 1) x += __shfl_xor(x, off);
    return x;
}

template <class POL, bool SPLIT>
__device__ __forceinline__ void p2p_leaves(const P2PArgs &a, const typename POL::Rec *__restrict__ parts,
                                           const POL &pol, double *red) {
    using Rec = typename POL::Rec;
    using T = typename POL::Real;
    double *fin = red + kRedRows * kP2PThreads;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Rec *__restrict__ targets = static_cast<const Rec *>(a.tparts);
    const size_t n = size_t(a.n);
    const int run = a.nleaf / int(gridDim.x);   // leaves of this workgroup
    const bool xcd = a.nleaf % 8 == 0 && gridDim.x % 8 == 0;
    const int first = xcd ? int(blockIdx.x & 7) * (a.nleaf >> 3) + int(blockIdx.x >> 3) * run : int(blockIdx.x) * run;
    const int nsh = int(gridDim.z) * kP2PWaves, sh = int(blockIdx.z) * kP2PWaves + wave;
    const T w = pol.scaled(T(a.w));
    for (int li = SPLIT ? 0 : wave; li < run; li += SPLIT ? 1 : kP2PWaves) {
        const int leaf = first + li;
        const int s0 = a.tstart[leaf], cnt = a.tstart[leaf + 1] - s0;
        if (cnt == 0) continue;
        // lane nb < 27: the neighbour's first source and the end of its sources in
        // the concatenated list
        int nb_js = 0, nb_end = 0;
        {
            LeafGeom L;
            L.side = 1 << a.level;
            L.cx = demorton(leaf, 0, a.level);
            L.cy = demorton(leaf, 1, a.level);
            L.cz = demorton(leaf, 2, a.level);
            int je = 0, dx, dy, dz;
            if (lane < 27 && !neighbour(a, L, lane, nb_js, je, dx, dy, dz)) nb_js = je = 0;
            nb_end = je - nb_js;
#pragma unroll
            for (int d = 1; d < 32; d <<= 1) {
                const int y = __shfl_up(nb_end, d, 64);
                if (lane >= d) nb_end += y;
            }
        }
        const int64_t total = __builtin_amdgcn_readlane(nb_end, 26);
        const int q0 = SPLIT ? int(total * sh / nsh) : 0, q1 = SPLIT ? int(total * (sh + 1) / nsh) : int(total);
        int piece = 0;
        for (int base = 0; base < cnt; ++piece) {
            const int E = piece_lanes(cnt - base);
            const int b0 = base;
            base += E;
            if (SPLIT && piece % int(gridDim.y) != int(blockIdx.y)) continue;
            const int t = lane & (E - 1), grp = lane / E, ng = 64 / E;
            const bool write = b0 + t < cnt && grp == 0;
            const int gi = s0 + (b0 + t < cnt ? b0 + t : b0);
            const Rec me = targets[gi];
            const T mx = pol.scaled(T(me.dx)), my = pol.scaled(T(me.dy)), mz = pol.scaled(T(me.dz));
            typename POL::Acc A;
            POL::clear(A);
            int c1 = 0;
            for (int nb = 0; nb < 27; ++nb) {
                const int c0 = c1;
                c1 = __builtin_amdgcn_readlane(nb_end, nb);
                const int p0 = SPLIT && q0 > c0 ? q0 : c0, p1 = SPLIT && q1 < c1 ? q1 : c1;
                if (p0 >= p1) continue;
                const int js = __builtin_amdgcn_readlane(nb_js, nb) + (p0 - c0), je = js + (p1 - p0);
                // x_i - x_j = (delta_i - d w) - delta_j, d = source - target cell offset
                const int dx = nb % 3 - 1, dy = (nb / 3) % 3 - 1, dz = nb / 9 - 1;
                const T tx = mx - T(dx) * w, ty = my - T(dy) * w, tz = mz - T(dz) * w;
                if (E == 64) pol.uniform(parts, js, je, tx, ty, tz, A);
                else pol.grouped(parts, js + grp, je, ng, tx, ty, tz, A);
            }
            auto sum = [&](auto kc) {   // SPLIT: the lane's share
                const double x = pol.template value<decltype(kc)::value>(A);
                return SPLIT ? x : group_sum(x, E);
            };
            const bool all = a.grad || a.dalpha;
            if constexpr (!SPLIT) {
                if (a.near) {
                    auto put = [&](auto kc) {
                        const double x = sum(kc);
                        if (write) a.near[size_t(decltype(kc)::value) * n + gi] = x;
                    };
                    for_rows(put, std::make_integer_sequence<int, 3>{});
                    if (all)
                        for_rows([&](auto kc) { put(IC<decltype(kc)::value + 3>{}); },
                                 std::make_integer_sequence<int, kNearRows - 3>{});
                } else {
                    double f[kNearRows];
                    for_rows([&](auto kc) { f[decltype(kc)::value] = sum(kc); },
                             std::make_integer_sequence<int, kNearRows>{});
                    finish(a, gi, write, [&](int r) { return f[r]; });
                }
            } else {
                // the waves' sums first, kRedRows rows a round, then the lane groups'
                auto round = [&](auto rc) {
                    wave_round<decltype(rc)::value>(red, sum, [&](int r, double x) {
                        x = group_sum(x, E);
                        if (!a.near) fin[r * 64 + lane] = x;
                        else if (write) a.near[(size_t(blockIdx.z) * kNearRows + r) * n + gi] = x;
                    });
                };
                round(IC<0>{});
                if (all)
                    for_rows([&](auto kc) { round(IC<decltype(kc)::value + 1>{}); },
                             std::make_integer_sequence<int, kNearRows / kRedRows - 1>{});
                if (!a.near && wave == 0) finish(a, gi, write, [&](int r) { return fin[64 * r + lane]; });
            }
        }
    }
}

inline int compute_units() {
    static const int ncu = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
            v = 256;
        return v;
    }();
    return ncu;
}


// blocks of 64 targets that a leaf holds on average, dealt over y; sources over z
inline int p2p_blocks(int nleaf, int ntarget, int slots) {
    return std::max(1, std::min(slots / nleaf, (ntarget / nleaf + 63) / 64));
}

// Leaves a workgroup takes: one where its waves split it (leaf counts are powers of
// 8, so at most 4096 leaves here, a few workgroups a compute unit), else one a wave.
struct P2PShape {
    bool split;
    dim3 grid;
    size_t smem;
};

// slots: workgroups the chip holds at once
inline P2PShape p2p_shape(const P2PArgs &a, int slots, int table_bytes) {
    P2PShape s;
    s.split = a.nleaf < kP2PSplitLeaves;
    const int run = s.split ? 1 : kP2PWaves;
    s.grid = dim3(unsigned(a.nleaf / run), unsigned(p2p_blocks(a.nleaf, a.n, slots)),
                  a.near ? unsigned(a.shares) : 1u);
    s.smem = size_t(table_bytes) + (s.split ? sizeof(double) * kRedDoubles : 0);
    return s;
}

}  // namespace
}  // namespace vmfmm
