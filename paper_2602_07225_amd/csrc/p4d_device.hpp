// Device helpers shared by the kernel files of the library.
#pragma once
#include "p4d_internal.hpp"

namespace p4d {

// Workgroup b of nb as dispatched round-robin over the 8 XCDs is mapped to a
// logical tile so that each XCD works on one contiguous range of tiles (its
// stencil halos then stay in that XCD's L2).
__device__ inline int xcd_block(int b, int nb)
{
    int q = nb >> 3, r = nb & 7;
    int x = b & 7, pos = b >> 3;
    int base = x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q;
    return base + pos;
}

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ inline double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Sum over a 256-thread workgroup; the result is valid in thread 0.
__device__ inline double block_sum(double v, double *lds /* >= 4 */)
{
    v = wave_sum(v);
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) lds[wv] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) r = (lds[0] + lds[1]) + (lds[2] + lds[3]);
    __syncthreads();
    return r;
}
__device__ inline double block_max(double v, double *lds)
{
    v = wave_max(v);
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) lds[wv] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) r = fmax(fmax(lds[0], lds[1]), fmax(lds[2], lds[3]));
    __syncthreads();
    return r;
}

// ---------------------------------------------------------------------------
// Krylov vectors with the particle part folded (see fgmres in p4d_api.hip):
// below the surface, the particle rows of every vector of a cycle are a
// multiple alpha of those of the cycle's first vector, whose sum of squares is
// sig2.  A vector is then its electrode-level rows, its surface rows (one per
// electrode node, phi_s order) and alpha.  The first vector is whole; FoldMap
// finds entry i of a folded vector in it (nm beyond every i: not folded).
// ---------------------------------------------------------------------------
__host__ __device__ inline FoldMap fold_map(const Geom &g)
{
    return FoldMap{g.Nm, g.Nm + g.nea, g.off_cs[0] + (long long)(g.nr[0] - 1) * g.nea - g.Nm,
                   g.off_cs[1] + (long long)(g.nr[1] - 1) * g.nec - g.Nm - g.nea};
}
__device__ inline long long fold_at(const FoldMap &M, long long i)
{
    return i < M.nm ? i : i + (i < M.na ? M.d0 : M.d1);
}
// Entry i of the vectors 0..nv-1 (vector q at V + q ldv, vector 0 at v0) to
// use(q, value), q ascending.  How they are loaded:
//  kBasisGroups  four vectors' loads to a (uniform) branch, the last ones'
//    repeated (to uses q >= nv, without effect), and no use in between, so that
//    they are all in flight together: dot products with 9..16 vectors of 0.9 M
//    entries 29.3 -> 20.7 us and the update 23.2 -> 17.9 against a test per
//    vector; 1.8 M entries 47 -> 34 and 40 -> 33.
//  kBasisEach  a test per vector, each load waited for: for few long vectors
//    (long_basis).
//  kBasisEights  groups of four, eight vectors used before the next are loaded:
//    for the dot products of more than 32 vectors, whose sums take 128
//    registers; with all loads ahead of the sums the kernel needed 256 and one
//    wave per SIMD.  48 vectors of 0.15 / 0.9 / 3.7 / 8 M entries: 36 / 118 /
//    291 / 564 us, all ahead 64 / 193 / 365 / 619, a test per vector 44 / 183 /
//    571 / 1164.
enum BasisLoads { kBasisGroups, kBasisEach, kBasisEights };
// waves per SIMD asked for: a load at a time wants all eight (at seven the
// 2048 workgroups of a long vector no longer run at once, half as fast again)
constexpr int basis_waves(int loads) { return loads == kBasisEach ? 8 : 1; }
template <int KMAX, int LOADS, typename Use>
__device__ inline void basis_row(const double *v0, const FoldMap &M, const double *V, long long ldv, int nv, long long i,
                                 Use use)
{
    const double *Vi = V + i;
    if constexpr (LOADS == kBasisEach) {
        use(0, v0[fold_at(M, i)]);
#pragma unroll
        for (int q = 1; q < KMAX; q++)
            if (q < nv) use(q, Vi[(long long)q * ldv]);
    } else {
        constexpr int C = LOADS == kBasisEights ? 8 : KMAX;
#pragma unroll
        for (int c = 0; c < KMAX; c += C) {
            if (LOADS == kBasisEights && c >= nv) continue;
            double v[C];
            if (c == 0) v[0] = v0[fold_at(M, i)];
#pragma unroll
            for (int g = c; g < c + C; g += 4) {
#pragma unroll
                for (int u = g ? 0 : 1; u < 4; u++) v[g - c + u] = 0.0;
                if ((g ? g : 1) < nv) {
#pragma unroll
                    for (int u = g ? 0 : 1; u < 4; u++)
                        v[g - c + u] = Vi[(long long)(g + u < nv ? g + u : nv - 1) * ldv];
                }
            }
#pragma unroll
            for (int q = 0; q < C; q++) use(c + q, v[q]);
        }
    }
}
// alpha of w = A P^-1 v_k before Gram-Schmidt (v_k's, normalized), or after
// its first pass
__device__ inline double fold_alpha(const double *alpha, const double *invbeta, int k, int pass)
{
    return pass == 0 ? alpha[k] * invbeta[k] : alpha[k + 1];
}
// the particle rows' part of w . V_q
__device__ inline double fold_dot(double aw, double aq, double sig2) { return aw * aq * sig2; }
// alpha after w -= sum_q c_q V_q, nv <= 64, by one whole wave (a lane per q)
__device__ inline double fold_update(double aw, const double *c, const double *alpha, int nv)
{
    const int q = threadIdx.x & 63;
    return aw - wave_sum(q < nv ? c[q] * alpha[q] : 0.0);
}

// workgroups of the pass over a cycle's first vector (two partial sums each)
__host__ __device__ inline int fold_nblk(const Geom &g)
{
    const long long b = (g.nnode + kBlock - 1) / kBlock;
    return (int)(b < 4096 ? b : 4096);
}
// its final sums by one workgroup: the norm, sig2, alpha_0 = 1 and 1 / norm
// (partial: the squares of the folded vector's rows and of the others)
__device__ inline void fold_final_block(const double *partial, int nblk, double *norm, double *sig2, double *alpha,
                                        double *invbeta, double *lds)
{
    double sy = 0.0, ss = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kBlock) {
        sy += partial[2 * b];
        ss += partial[2 * b + 1];
    }
    sy = block_sum(sy, lds);
    ss = block_sum(ss, lds);
    if (threadIdx.x == 0) {
        const double bt = sqrt(sy + ss);
        *norm = bt;
        *sig2 = ss;
        *alpha = 1.0;
        if (invbeta) *invbeta = bt > 0.0 ? 1.0 / bt : 0.0;
    }
}

__host__ __device__ constexpr int popc3(int v) { return (v & 1) + ((v >> 1) & 1) + ((v >> 2) & 1); }
__host__ __device__ constexpr int nb_index(int dx, int dy, int dz)
{
    return (dx + 1) + 3 * (dy + 1) + 9 * (dz + 1);
}

// Q1 element sums at one node.  c[e], e = ex | ey<<1 | ez<<2, is the
// coefficient of the element spanning node offsets ex-1..ex (etc.); X holds
// the 27 neighbour values.  Reference stiffness on the unit cube: 1/3 on the
// diagonal, 0 between corners differing in one coordinate, -1/12 otherwise.
// Its rows sum to zero, so it is applied to differences x_b - x_a: constants
// cancel exactly, which keeps near-null modes accurate in FP32.
template <typename R>
__device__ inline R q1_stiff(const R c[8], const R X[27])
{
    R acc = R(0);
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int ex = e & 1, ey = (e >> 1) & 1, ez = (e >> 2) & 1;
        const int a = (1 - ex) | ((1 - ey) << 1) | ((1 - ez) << 2);
        R far = R(0);
#pragma unroll
        for (int bb = 0; bb < 8; bb++) {
            if (popc3(a ^ bb) >= 2)
                far += X[13] - X[nb_index(ex - 1 + (bb & 1), ey - 1 + ((bb >> 1) & 1),
                                          ez - 1 + ((bb >> 2) & 1))];
        }
        acc += c[e] * far;
    }
    return acc * R(1.0 / 12.0);
}

// The same for box elements: kw[p] weighs the difference to the corner that
// differs in the axes of bit pattern p (kw[0], the diagonal, is not used:
// rows sum to zero).  With kw = {., 0, 0, 1/12, 0, 1/12, 1/12, 1/12} it is
// q1_stiff.
template <typename R>
__device__ inline R q1_stiff_w(const R c[8], const R X[27], const double kw[8])
{
    R acc = R(0);
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int ex = e & 1, ey = (e >> 1) & 1, ez = (e >> 2) & 1;
        const int a = (1 - ex) | ((1 - ey) << 1) | ((1 - ez) << 2);
        R part = R(0);
#pragma unroll
        for (int bb = 0; bb < 8; bb++) {
            if (bb == a) continue;
            part += R(kw[a ^ bb]) * (X[13] - X[nb_index(ex - 1 + (bb & 1), ey - 1 + ((bb >> 1) & 1),
                                                      ez - 1 + ((bb >> 2) & 1))]);
        }
        acc += c[e] * part;
    }
    return acc;
}

// Reference mass on the unit cube: (8, 4, 2, 1)/216 by the number of
// differing coordinates.
template <typename R>
__device__ inline R q1_mass(const R c[8], const R X[27])
{
    R acc = R(0);
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int ex = e & 1, ey = (e >> 1) & 1, ez = (e >> 2) & 1;
        const int a = (1 - ex) | ((1 - ey) << 1) | ((1 - ez) << 2);
        R part = R(0);
#pragma unroll
        for (int bb = 0; bb < 8; bb++) {
            const int d = popc3(a ^ bb);
            const R w = d == 0 ? R(8.0 / 216.0) : d == 1 ? R(4.0 / 216.0)
                                                         : d == 2 ? R(2.0 / 216.0) : R(1.0 / 216.0);
            part += w * X[nb_index(ex - 1 + (bb & 1), ey - 1 + ((bb >> 1) & 1),
                                   ez - 1 + ((bb >> 2) & 1))];
        }
        acc += c[e] * part;
    }
    return acc;
}

}  // namespace p4d
