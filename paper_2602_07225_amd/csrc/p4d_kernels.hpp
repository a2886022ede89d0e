// Block-level device functions of the operator and the preconditioner.  The
// single-cell kernels (operator.hip, radial.hip, mg.hip) and the batched stage
// kernels (batch.hip, one launch per stage depth over work lists spanning all
// cells) call the same functions, each for one workgroup-sized unit of work
// given by an explicit block or tile index.
#pragma once
#include "p4d_device.hpp"

namespace p4d {

// ---------------------------------------------------------------------------
// 1D transfer helpers for 'even indices plus the last' coarsening of n points
// ---------------------------------------------------------------------------
__host__ __device__ inline int coarse_n(int n) { return n <= 2 ? n : n / 2 + 1; }

// coarse points (and weights) that fine point i interpolates from
__device__ inline int coarse_of(int n, int i, int I[2], double w[2])
{
    // (an unused second slot repeats the first point with weight 0)
    if (n <= 2) { I[0] = I[1] = i; w[0] = 1.0; w[1] = 0.0; return 1; }
    if (!(i & 1)) { I[0] = I[1] = i >> 1; w[0] = 1.0; w[1] = 0.0; return 1; }
    if (i == n - 1) { I[0] = I[1] = n / 2; w[0] = 1.0; w[1] = 0.0; return 1; }
    I[0] = (i - 1) >> 1; w[0] = 0.5;
    I[1] = (i + 1) >> 1; w[1] = 0.5;
    return 2;
}
// fine points (and weights) that interpolate from coarse point I, in the
// order: the coincident point, its odd left neighbour, its odd right
// neighbour; unused slots repeat the coincident point with weight 0
// (selects instead of a running index keep the arrays in registers)
__device__ inline int fine_of(int n, int I, int f[3], double w[3])
{
    if (n <= 2) {
        f[0] = f[1] = f[2] = I;
        w[0] = 1.0; w[1] = w[2] = 0.0;
        return 1;
    }
    const int nc = n / 2 + 1;
    const int c = (I == nc - 1) ? n - 1 : 2 * I;
    const bool lft = c - 1 >= 0 && ((c - 1) & 1) && c - 1 != n - 1;
    const bool rgt = c + 1 <= n - 1 && ((c + 1) & 1) && c + 1 != n - 1;
    f[0] = c; w[0] = 1.0;
    f[1] = lft ? c - 1 : (rgt ? c + 1 : c);
    w[1] = (lft || rgt) ? 0.5 : 0.0;
    f[2] = (lft && rgt) ? c + 1 : c;
    w[2] = (lft && rgt) ? 0.5 : 0.0;
    return 1 + (int)lft + (int)rgt;
}

template <typename B>
__device__ inline int find_box(const B &bt, int b)
{
    int q = 0;
#pragma unroll
    for (int t = 1; t < 4; t++)
        if (t < bt.nbox && b >= bt.a[t].blk0) q = t;
    return q;
}

// ---------------------------------------------------------------------------
// Level-0 smoother, 2.5D tiled.  A workgroup owns a TX x TY tile of an x-y
// plane and marches through a chunk of CZ node layers; three planes of x
// (with a one-node halo) and two layers of element coefficients sit in LDS
// rings, so every value is read from memory once per tile and the 27-point
// neighbourhood comes from LDS.  TX in {16, 32, 64}, TY = 256 / TX.
// ---------------------------------------------------------------------------
constexpr int kXpLds = 396;   // largest plane with halo: 66 x 6
constexpr int kCkLds = 325;   // largest element tile: 65 x 5
struct Smooth0Lds {
    double xp[3][kXpLds];
    double ck[2][kCkLds];
};

__host__ __device__ inline int smooth0_box_tiles(int nx, int ny, int nz, int TX, int CZ)
{
    const int TY = kBlock / TX;
    return ((nx + TX - 1) / TX) * ((ny + TY - 1) / TY) * ((nz + CZ - 1) / CZ);
}

// Q1 stiffness at a node: box-element weights g.kw in the general (GEN)
// instantiations, the cube stencil otherwise
template <bool GEN, typename R>
__device__ inline R stiff_of(const Geom &g, const R c[8], const R X[27])
{
    if (GEN) return q1_stiff_w(c, X, g.kw);
    return q1_stiff(c, X);
}

// The cube stencil as the level-0 smoother evaluates it.  The rows sum to
// zero, so the node's row is (4 x_i sum_e c_e - sum_e c_e F_e) / 12, with
// F_e the sum of x over the four corners of element e that differ from the
// node in at least two axes.  That is ~41 FP64 operations per node against
// ~72 for the difference form; the rounding differs by a few ulps of
// |x_i| sum_e c_e, which is far below what a smoothing step resolves.
template <typename R>
__device__ inline R q1_stiff_sum(const R c[8], const R X[27])
{
    R acc = R(0), cs = R(0);
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int ex = e & 1, ey = (e >> 1) & 1, ez = (e >> 2) & 1;
        const int a = (1 - ex) | ((1 - ey) << 1) | ((1 - ez) << 2);
        R far = R(0);
        bool first = true;
#pragma unroll
        for (int bb = 0; bb < 8; bb++) {
            if (popc3(a ^ bb) < 2) continue;
            const R v = X[nb_index(ex - 1 + (bb & 1), ey - 1 + ((bb >> 1) & 1), ez - 1 + ((bb >> 2) & 1))];
            far = first ? v : far + v;
            first = false;
        }
        acc = e == 0 ? c[e] * far : acc + c[e] * far;
        cs = e == 0 ? c[e] : cs + c[e];
    }
    return (R(4) * X[13] * cs - acc) * R(1.0 / 12.0);
}

// MEH: the storage of the mass box per element (g.meh) and the box-element
// stiffness weights (a separate instantiation keeps the per-material cube
// one free of their registers)
template <typename T, bool RESID_ONLY, bool MEH = false>
__device__ inline void smooth0_tile(const Geom &g, const LevelArgs<T> &A, int tile, int TX, int CZ,
                                    Smooth0Lds &L)
{
    const int TY = kBlock / TX;
    const int PX = TX + 2, PY = TY + 2;
    const int EX = TX + 1, EY = TY + 1;
    const int ntx = (A.nx + TX - 1) / TX, nty = (A.ny + TY - 1) / TY;
    const int tix = tile % ntx, tiy = (tile / ntx) % nty, tch = tile / (ntx * nty);
    const int i0 = tix * TX, j0 = tiy * TY, k0l = tch * CZ;
    const int k1l = k0l + CZ < A.nz ? k0l + CZ : A.nz;
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    const int i = i0 + tx, j = j0 + ty;
    const bool own = i < A.nx && j < A.ny;
    const int planeN = A.nx * A.ny;
    // elements on either side of the node in x and y (the box spans the
    // whole node plane)
    const bool inx0 = i > 0, inx1 = i < g.nx - 1, iny0 = j > 0, iny1 = j < g.ny - 1;

    // One plane of x with its halo (PX*PY <= 2*kBlock values) and one layer
    // of element coefficients (EX*EY <= 2*kBlock) per workgroup: each thread
    // holds at most two of each.  They are fetched into registers one layer
    // ahead and written to LDS after the layer that used the slot is done,
    // so the global loads overlap the arithmetic of the previous layer.
    double px[2], pc[2];
    auto fetch_plane_to = [&](int kl, double v[2]) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            const int ii = i0 - 1 + q % PX, jj = j0 - 1 + q / PX;
            const bool ok = q < PX * PY && kl >= 0 && kl < A.nz && ii >= 0 && ii < A.nx && jj >= 0 &&
                            jj < A.ny;
            v[h] = ok ? A.xin[ii + A.nx * (jj + A.ny * kl)] : 0.0;
        }
    };
    auto store_plane_from = [&](int slot, const double v[2]) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            if (q < PX * PY) L.xp[slot][q] = v[h];
        }
    };
    auto fetch_elems_to = [&](int kl, double v[2]) {
        const int ek = kl + A.k0;
        const bool lay = ek >= A.ek_lo && ek <= A.ek_hi;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            const int ei = i0 - 1 + q % EX, ej = j0 - 1 + q / EX;
            const bool ok = q < EX * EY && lay && ei >= 0 && ei < g.nx - 1 && ej >= 0 && ej < g.ny - 1;
            v[h] = ok ? A.cK[ei + (long long)(g.nx - 1) * (ej + (long long)(g.ny - 1) * ek)] : 0.0;
        }
    };
    auto store_elems_from = [&](int slot, const double v[2]) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            if (q < EX * EY) L.ck[slot][q] = v[h];
        }
    };
    auto fetch_plane = [&](int kl) { fetch_plane_to(kl, px); };
    auto store_plane = [&](int slot) { store_plane_from(slot, px); };
    auto fetch_elems = [&](int kl) { fetch_elems_to(kl, pc); };
    auto store_elems = [&](int slot) { store_elems_from(slot, pc); };
    // per-node data of a layer (right-hand side, reaction diagonal, inverse
    // diagonal, previous direction), also fetched one layer ahead
    double nb[4] = {0.0, 0.0, 0.0, 0.0};
    auto fetch_node = [&](int kl) {
        const int n = i + A.nx * j + planeN * kl;
        if (own) {
            nb[0] = (double)A.b[n];
            nb[1] = (double)A.dcorr[n];
            if (!RESID_ONLY) {
                nb[2] = (double)A.invd[n];
                if (A.c1 != 0.0 && !A.din_x) nb[3] = (double)A.din[n];
            }
        }
    };
    {   // prologue: every load of the first layer is issued before any of
        // them is stored, so the tile waits for one memory latency, not four
        double p0[2], p1[2], e0[2];
        fetch_plane_to(k0l - 1, p0);
        fetch_plane_to(k0l, p1);
        fetch_elems_to(k0l - 1, e0);
        fetch_plane(k0l + 1);
        fetch_elems(k0l);
        fetch_node(k0l);
        store_plane_from((k0l + 2) % 3, p0);
        store_plane_from(k0l % 3, p1);
        store_elems_from((k0l + 1) & 1, e0);
    }
    for (int kl = k0l; kl < k1l; kl++) {
        store_plane((kl + 1) % 3);
        store_elems(kl & 1);
        const int n = i + A.nx * j + planeN * kl;
        const double bn = nb[0], dcn = nb[1], idn = nb[2], dnn = nb[3];
        __syncthreads();
        if (kl + 1 < k1l) {
            fetch_plane(kl + 2);
            fetch_elems(kl + 1);
            fetch_node(kl + 1);
        }
        if (own) {
            double X[27];
#pragma unroll
            for (int dz = -1; dz <= 1; dz++) {
                const double *P = L.xp[(kl + dz + 3) % 3];
#pragma unroll
                for (int dy = -1; dy <= 1; dy++)
#pragma unroll
                    for (int dx = -1; dx <= 1; dx++)
                        X[nb_index(dx, dy, dz)] = P[(tx + 1 + dx) + PX * (ty + 1 + dy)];
            }
            double cK[8], cM[8];
            const int k = kl + A.k0;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const int ex = e & 1, ey = (e >> 1) & 1, ez = (e >> 2) & 1;
                cK[e] = L.ck[(kl - 1 + ez) & 1][(tx + ex) + EX * (ty + ey)];
                // storage of the elements inside the box, whatever their
                // stiffness coefficient (which may be zero)
                const int ek = k - 1 + ez;
                const bool in = A.mass && (ex ? inx1 : inx0) && (ey ? iny1 : iny0) &&
                                ek >= A.ek_lo && ek <= A.ek_hi;
                if (MEH) {
                    const int ei = i - 1 + ex, ej = j - 1 + ey;
                    cM[e] = in ? elem_storage(g, ei + (long long)(g.nx - 1) * (ej + (long long)(g.ny - 1) * ek), ek)
                               : 0.0;
                } else {
                    cM[e] = in ? (elem_mat(g, ek) >= 0 ? g.mass_elec : g.mass_sep) : 0.0;
                }
            }
            double Sx = (MEH ? q1_stiff_w(cK, X, g.kw) : q1_stiff_sum(cK, X)) + dcn * X[13];
            if (A.mass) Sx += q1_mass(cM, X);
            const double r = bn - Sx;
            if (RESID_ONLY) {
                A.rout[n] = (T)r;
            } else {
                double d = A.c2 * idn * r;
                if (A.c1 != 0.0) d += A.c1 * (A.din_x ? X[13] : dnn);
                A.xout[n] = X[13] + d;
                if (A.dout) A.dout[n] = (T)d;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Levels >= 1: Galerkin stencil of a symmetric operator, stored by its upper
// half in difference form: slot 0 holds the row sum, slot 1 + u the coupling
// to the neighbour at stencil offset 14 + u; the coupling to a neighbour at
// a lower offset o is that neighbour's coupling at offset 26 - o.
//   S x = rowsum x_i + sum_{j != i} s_ij (x_j - x_i)
// ---------------------------------------------------------------------------
// S x at a node from its 27 couplings (zero to a missing neighbour, whose x
// may then be any finite value) and neighbourhood
template <typename T>
__device__ inline double stencil_row(const T sv[27], const double xv[27])
{
    const double xc = xv[13];
    double Sx = (double)sv[13] * xc;
#pragma unroll
    for (int o = 0; o < 27; o++) {
        if (o == 13) continue;
        Sx += (double)sv[o] * (xv[o] - xc);
    }
    return Sx;
}
// which neighbours of node (i, j, k) lie on an nx x ny x nz grid: bit d + 1
// per axis and offset d, and the answer for stencil offset o (0 or 1), formed
// without branches
struct NbMask {
    unsigned x, y, z;
    __device__ NbMask(int i, int j, int k, int nx, int ny, int nz)
        : x((i > 0 ? 1u : 0u) | 2u | (i < nx - 1 ? 4u : 0u)), y((j > 0 ? 1u : 0u) | 2u | (j < ny - 1 ? 4u : 0u)),
          z((k > 0 ? 1u : 0u) | 2u | (k < nz - 1 ? 4u : 0u))
    {
    }
    __device__ int has(int o) const { return (x >> (o % 3)) & (y >> (o / 3 % 3)) & (z >> (o / 9)) & 1u; }
};
// one Chebyshev step from the residual r: the direction (dprev: the previous
// one, used if c1 != 0)
__device__ inline double cheb_dir(double c1, double c2, double invd, double r, double dprev)
{
    double d = c2 * invd * r;
    if (c1 != 0.0) d += c1 * dprev;
    return d;
}

template <typename T, bool RESID_ONLY>
__device__ inline void smooth_block(const LevelArgs<T> &A, int blk)
{
    const int n = blk * kBlock + threadIdx.x;
    if (n >= A.n) return;
    const int i = n % A.nx, t = n / A.nx;
    const NbMask M(i, t % A.ny, t / A.ny, A.nx, A.ny, A.nz);
    // all coefficients and neighbours are loaded before any arithmetic (a
    // missing neighbour's index is clamped to the node, its coupling dropped),
    // so the loads are in flight together
    T sv[27];
    double xv[27];
#pragma unroll
    for (int o = 0; o < 27; o++) {
        const int h = M.has(o), nbr = n + (((o % 3 - 1) + A.nx * ((o / 3) % 3 - 1 + A.ny * (o / 9 - 1))) & -h);
        xv[o] = A.xin[nbr];
        const T v = o >= 13 ? A.S[(long long)(o - 13) * A.n + n] : A.S[(long long)(13 - o) * A.n + nbr];
        sv[o] = h ? v : T(0);
    }
    const double xc = xv[13];
    const double r = (double)A.b[n] - stencil_row(sv, xv);
    if (RESID_ONLY) {
        A.rout[n] = (T)r;
        return;
    }
    const double d = cheb_dir(A.c1, A.c2, (double)A.invd[n], r,
                              A.c1 != 0.0 ? (A.din_x ? xc : (double)A.din[n]) : 0.0);
    A.xout[n] = xc + d;
    if (A.dout) A.dout[n] = (T)d;
}

// (P^T r_f) at coarse node n
template <typename Ptr>
__device__ inline double restrict_value(int fx, int fy, int fz, int cx, int cy, int cz, int n, Ptr rf)
{
    const int I = n % cx, t = n / cx;
    const int J = t % cy, K = t / cy;
    int fi[3], fj[3], fk[3];
    double wi[3], wj[3], wk[3];
    fine_of(fx, I, fi, wi);
    fine_of(fy, J, fj, wj);
    fine_of(cz == fz ? 1 : fz, K, fk, wk);   // (z kept: identity)
    // all 27 slots, without tests: an unused slot reads a point that a used
    // slot reads too and adds an exact zero to a sum that starts at +0 (and
    // so never holds -0), leaving it as it is bit for bit; unguarded, the
    // loads are all in flight at once
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < 3; c++) {
#pragma unroll
        for (int bq = 0; bq < 3; bq++) {
            const int row = fx * (fj[bq] + fy * fk[c]);
            double part = 0.0;
#pragma unroll
            for (int a = 0; a < 3; a++) part += wi[a] * (double)rf[row + fi[a]];
            acc += wj[bq] * wk[c] * part;
        }
    }
    return acc;
}

// b_c = P^T r_f; also the first Chebyshev iterate x_c1 = c2 D_c^-1 b_c
template <typename T>
__device__ inline void restrict_block(const TransferArgs<T> &A, int blk)
{
    const int nc = A.cx * A.cy * A.cz;
    const int n = blk * kBlock + threadIdx.x;
    if (n >= nc) return;
    // issued with the residual loads (after the store below it would wait
    // for them first)
    const double idc = A.xc1 ? (double)A.invdc[n] : 0.0;
    const T bc = (T)restrict_value(A.fx, A.fy, A.fz, A.cx, A.cy, A.cz, n, A.rf);
    A.bc[n] = bc;
    if (A.xc1) A.xc1[n] = A.c2c * idc * (double)bc;
}

// (P x_c) at fine node (i, j, k); coarse node (I, J, K) at xc[I + sy J + sz K]
template <typename Ptr>
__device__ inline double prolong_value(int fx, int fy, int fz, bool keepz, int i, int j, int k, Ptr xc, int sy, int sz)
{
    int Ci[2], Cj[2], Ck[2];
    double wi[2], wj[2], wk[2];
    coarse_of(fx, i, Ci, wi);
    coarse_of(fy, j, Cj, wj);
    coarse_of(keepz ? 1 : fz, k, Ck, wk);
    // all 8 slots, without tests (an unused slot adds an exact zero; see
    // restrict_block)
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < 2; c++) {
#pragma unroll
        for (int bq = 0; bq < 2; bq++) {
            const int row = sy * Cj[bq] + sz * Ck[c];
            double part = 0.0;
#pragma unroll
            for (int a = 0; a < 2; a++) part += wi[a] * xc[row + Ci[a]];
            acc += wj[bq] * wk[c] * part;
        }
    }
    return acc;
}

// x_f += P x_c
template <typename T>
__device__ inline void prolong_block(const TransferArgs<T> &A, int blk)
{
    const int nf = A.fx * A.fy * A.fz;
    const int n = blk * kBlock + threadIdx.x;
    if (n >= nf) return;
    const int i = n % A.fx, t = n / A.fx;
    const int j = t % A.fy, k = t / A.fy;
    A.xf[n] += prolong_value(A.fx, A.fy, A.fz, A.cz == A.fz, i, j, k, A.xc, A.cx, A.cx * A.cy);
}

// Prolongation and the first post-smoothing step of small levels >= 1 in one
// pass: a workgroup forms x + P x_c on a tile of 8 x 8 x 4 nodes and the nodes
// around it in LDS, a thread each, and smooths the tile; the arithmetic is
// that of the two stages, bit for bit.  The two launches are bound by launch
// and latency on small levels: 3.2 to 4.0 + 4.3 to 4.6 us up to 100
// workgroups, 5.1 to 5.8 in one; with the two rounds of workgroups that the
// chip takes (a workgroup a CU, 119 registers and ten waves) 4 + 4.8 and 7.7;
// with three 5 + 6.5 and 14.0, since 344 of 600 nodes are formed once more by
// each neighbour: kFineTiles ends at two.  (The residual with the restriction
// in the same way took 6.9 to 9.4 us against 8: left apart.)
constexpr int kFineTiles = 512;
constexpr int kFineX = 8, kFineY = 8, kFineZ = 4;
constexpr int kFineThreads = 640;     // a node with halo each, the first 256 smooth
constexpr int kFineHalo = (kFineX + 2) * (kFineY + 2) * (kFineZ + 2);
__host__ __device__ inline int fine_tiles(int nx, int ny, int nz)
{
    return ((nx + kFineX - 1) / kFineX) * ((ny + kFineY - 1) / kFineY) * ((nz + kFineZ - 1) / kFineZ);
}
template <typename T>
__device__ inline void prolong_smooth_block(const LevelArgs<T> &A, const TransferArgs<T> &R, int tile, double *lds)
{
    const int tx = (A.nx + kFineX - 1) / kFineX, ty = (A.ny + kFineY - 1) / kFineY;
    const int i0 = tile % tx * kFineX, j0 = tile / tx % ty * kFineY, k0 = tile / tx / ty * kFineZ;
    const int i = i0 + threadIdx.x % kFineX, j = j0 + threadIdx.x / kFineX % kFineY,
              k = k0 + threadIdx.x / (kFineX * kFineY);
    const bool own = threadIdx.x < kFineX * kFineY * kFineZ && i < A.nx && j < A.ny && k < A.nz;
    const int n = own ? i + A.nx * (j + A.ny * k) : 0;
    const NbMask M(i, j, k, A.nx, A.ny, A.nz);
    // the couplings are on their way while x is formed
    T sv[27];
    if (own) {
#pragma unroll
        for (int o = 0; o < 27; o++) {
            const int h = M.has(o), nbr = n + (((o % 3 - 1) + A.nx * ((o / 3) % 3 - 1 + A.ny * (o / 9 - 1))) & -h);
            sv[o] = o >= 13 ? A.S[(long long)(o - 13) * A.n + n] : A.S[(long long)(13 - o) * A.n + nbr];
        }
    }
    const double bn = own ? (double)A.b[n] : 0.0, idn = own ? (double)A.invd[n] : 0.0;
    constexpr int HX = kFineX + 2, HY = kFineY + 2;
    const int q = threadIdx.x;
    if (q < kFineHalo) {
        const int ii = i0 - 1 + q % HX, jj = j0 - 1 + q / HX % HY, kk = k0 - 1 + q / (HX * HY);
        double v = 0.0;
        if (ii >= 0 && ii < A.nx && jj >= 0 && jj < A.ny && kk >= 0 && kk < A.nz) {
            v = A.xin[ii + A.nx * (jj + A.ny * kk)];
            v += prolong_value(A.nx, A.ny, A.nz, R.cz == A.nz, ii, jj, kk, R.xc, R.cx, R.cx * R.cy);
        }
        lds[q] = v;
    }
    __syncthreads();
    if (!own) return;
    double xv[27];
    const double *P = lds + (i - i0 + 1) + HX * ((j - j0 + 1) + HY * (k - k0 + 1));
#pragma unroll
    for (int o = 0; o < 27; o++) {
        xv[o] = P[(o % 3 - 1) + HX * ((o / 3) % 3 - 1 + HY * (o / 9 - 1))];
        sv[o] = M.has(o) ? sv[o] : T(0);
    }
    const double d = cheb_dir(A.c1, A.c2, idn, bn - stencil_row(sv, xv), 0.0);   // c1 = 0 in the first step
    A.xout[n] = xv[13] + d;
    if (A.dout) A.dout[n] = (T)d;
}

// Coarsest level, 64 rows of x = A^-1 b per workgroup (FP64); the 4 waves
// split the columns, then add up.
struct CoarseLds {
    double bl[1024];
    double part[4][64];
};
template <typename T>
__device__ inline void coarse_block(const CoarseArgs<T> &A, int rowblk, CoarseLds &L)
{
    const int n = A.n;
    for (int q = threadIdx.x; q < n; q += kBlock) L.bl[q] = (double)A.b[q];
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int row = rowblk * 64 + lane;
    double acc = 0.0;
    if (row < n) {
#pragma unroll 4
        for (int c = w; c < n; c += 4) acc += A.Ainv[(long long)c * n + row] * L.bl[c];
    }
    L.part[w][lane] = acc;
    __syncthreads();
    if (w == 0 && row < n)
        A.x[row] = (L.part[0][lane] + L.part[1][lane]) + (L.part[2][lane] + L.part[3][lane]);
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Particle blocks (Sec. 4.2: one tridiagonal system per point, inverted
// exactly).  A_ss,j = T0 + Gamma s_j e_N e_N^T shares the LU of T0; only the
// last pivot depends on the node.
// ---------------------------------------------------------------------------
// A radial table read through the constant address space: loads from a
// wave-uniform address become scalar loads (the tables do not change while
// a kernel runs)
typedef __attribute__((address_space(4))) const RadialTab ConstTab;

struct RadArgs {
    const RadialTab *tabs;
    const double *gg, *ss, *ee, *mm, *om;
    void *b0;            // T, macro layout
    double *x1;          // first Chebyshev iterate of each box
    const void *invd0;   // T
    double c2box[4];
    const double *x0[4]; // final level-0 iterates per box (rad_back)
};

// The surface rows of a folded vector at one electrode node, scaled: ap the
// scaled alpha, e what the surface row has beyond ap times the first vector's
// (rounding, as long as P solves the particle rows exactly)
struct FoldNode {
    double ap, e;
};
__device__ inline FoldNode fold_node(const Geom &g, const FoldVec &F, long long je)
{
    const double sc = *F.scale;
    FoldNode n{*F.alpha * sc, 0.0};
    if (F.vs) n.e = F.vs[je] * sc - n.ap * F.v0[fold_at(fold_map(g), g.Nm + je)];
    return n;
}
// row q of z_s,j = A_ss,j^-1 (r_s,j - delta_j e_N) for a folded r: u is row q
// of A_ss,j^-1 s_j, t that of T0^-1 e_N, eo = e omega_j, dw = delta_j omega_j
__device__ inline double fold_row(double ap, double u, double eo, double dw, double t)
{
    const double zn = ap * u + eo * t;
    return zn - dw * t;
}
// delta_j of A_sy z (transposed A_ys^T z)
template <bool TRANS, typename Tab>
__device__ inline double fold_delta(const Geom &g, const Tab &T, bool dir, double m, double gj, double sj, double ej,
                                    double zps, double zpe, double zce)
{
    if (!TRANS) return T.Gamma * ((dir ? 0.0 : gj) * zps - gj * zpe + ej * zce);
    return sj * ((dir ? 0.0 : m) * zps - m * zpe - g.tc * m * zce);
}

// zeta_j = (A_ss,j^-1 r_s,j)_N; r~_y = r_y - a_y s_j zeta_j (transposed:
// r_y - Gamma b_y zeta_j); written in precision T with the first Chebyshev
// iterate of each box.  SCHUR 0: r~_y = r_y; 1: zeta_j by elimination; 2: a
// folded vector F.
template <typename T, int NRMAX, bool TRANS, int SCHUR>
__device__ inline void rad_fwd_block(const Geom &g, const RadArgs &R, const double *r, double rscale,
                                     int blk, const FoldVec &F = FoldVec{})
{
    const long long n = (long long)blk * kBlock + threadIdx.x;
    if (n >= g.nnode) return;
    T *b0 = (T *)R.b0;
    const T *invd0 = (const T *)R.invd0;
    const int k = (int)(n / ((long long)g.nx * g.ny));
    double rpe = r[g.off_pe + n] * rscale;
    double rce = r[g.off_ce + n] * rscale;
    // every load is issued before the first store (a load after a store of
    // a computed value would wait for that computation's loads first)
    const double idpe = (double)invd0[g.off_pe + n], idce = (double)invd0[g.off_ce + n];
    const int el = node_mat(g, k);
    if (el >= 0) {
        const long long base = el == 0 ? 0 : g.nea;
        const long long klo = el == 0 ? 0 : g.na + g.ns;
        const long long je = base + n - klo * g.nx * g.ny;
        const bool dir = (k == 0);
        double rps = r[je] * rscale;
        const double idps = dir ? 0.0 : (double)invd0[je];
        // r~ from zeta_j; Gam is only used transposed
        auto couple = [&](double zeta, double Gam, double sj) {
            const double m = R.mm[je];
            if (!TRANS) {   // a_y s_j zeta, a_y = (m, -m, -tc m)
                const double f = sj * zeta;
                if (!dir) rps -= m * f;
                rpe += m * f;
                rce += g.tc * m * f;
            } else {        // Gamma b_y zeta, b_y = (g, -g, e)
                const double f = Gam * zeta;
                const double gj = R.gg[je];
                if (!dir) rps -= gj * f;
                rpe += gj * f;
                rce -= R.ee[je] * f;
            }
        };
        if (SCHUR == 2) {
            const double tN = el == 0 ? R.tabs[0].tau0 : R.tabs[1].tau0;
            const FoldNode fn = fold_node(g, F, je);
            couple(fold_row(fn.ap, F.u0[je], fn.e * R.om[je], 0.0, tN), el == 0 ? R.tabs[0].Gamma : R.tabs[1].Gamma,
                   R.ss[je]);
        } else if (SCHUR) {
            auto elim = [&](const auto &Tb) {
                const int N = Tb.N;
                const long long nn = el == 0 ? g.nea : g.nec;
                const double *rs = r + (el == 0 ? g.off_cs[0] : g.off_cs[1]) + (je - base);
                // all radial values first (indices clamped to the last point), so
                // the loads are in flight together
                double rv[NRMAX];
#pragma unroll
                for (int q = 0; q < NRMAX; q++) rv[q] = rs[(long long)(q < N ? q : N - 1) * nn];
                T y = (T)(rv[0] * rscale);
#pragma unroll
                for (int q = 1; q < NRMAX; q++) {
                    if (q < N) {
                        const T lq = (T)(TRANS ? Tb.lT[q] : Tb.l[q]);
                        y = (T)(rv[q] * rscale) - lq * y;
                    }
                }
                const double sj = R.ss[je];
                const T pivN = (T)(Tb.piv[N - 1] + Tb.Gamma * sj);
                couple((double)(y / pivN), Tb.Gamma, sj);
            };
            // the tables of the node's electrode: through a wave-uniform pointer
            // in the constant address space (scalar loads) when the whole wave
            // lies in one electrode, per lane otherwise
            const int elw = __builtin_amdgcn_readfirstlane(el);
            if (__builtin_amdgcn_ballot_w64(el != elw) == 0) elim(*(const ConstTab *)(R.tabs + elw));
            else elim(R.tabs[el]);
        }
        const T bps = (T)rps;
        b0[je] = bps;
        if (!dir) R.x1[je] = (el == 0 ? R.c2box[0] : R.c2box[1]) * idps * (double)bps;
    }
    const T bpe = (T)rpe, bce = (T)rce;
    b0[g.off_pe + n] = bpe;
    b0[g.off_ce + n] = bce;
    R.x1[g.off_pe + n] = R.c2box[2] * idpe * (double)bpe;
    R.x1[g.off_ce + n] = R.c2box[3] * idce * (double)bce;
}

// z_s,j = A_ss,j^-1 r_s,j - delta_j A_ss,j^-1 e_N, and by Sherman-Morrison
// A_ss,j^-1 e_N = omega_j T0^-1 e_N: the elimination in precision T only
// sees r_s, while delta_j = Gamma b_y . z_y (transposed s_j a_y . z_y),
// which carries the large near-null part of z_y, is applied in FP64.
template <typename T, typename TZ, int NRMAX, bool TRANS, bool SCHUR>
__device__ inline void rad_back_block(const Geom &g, const RadArgs &R, const double *r, double rscale,
                                      TZ *z, int blk)
{
    const long long n = (long long)blk * kBlock + threadIdx.x;
    if (n >= g.nnode) return;
    const int k = (int)(n / ((long long)g.nx * g.ny));
    const int el = node_mat(g, k);
    const double zpe = R.x0[2][g.off_pe + n];
    const double zce = R.x0[3][g.off_ce + n];
    if (el < 0) {
        z[g.off_pe + n] = (TZ)zpe;
        z[g.off_ce + n] = (TZ)zce;
        return;
    }
    const long long base = el == 0 ? 0 : g.nea;
    const long long klo = el == 0 ? 0 : g.na + g.ns;
    const long long je = base + n - klo * g.nx * g.ny;
    const bool dir = (k == 0);
    const double zps = dir ? r[je] * rscale : (el == 0 ? R.x0[0] : R.x0[1])[je];
    auto solve = [&](const auto &Tb) {
        const int N = Tb.N;
        const long long nn = el == 0 ? g.nea : g.nec;
        const double *rs = r + (el == 0 ? g.off_cs[0] : g.off_cs[1]) + (je - base);
        TZ *zs = z + (el == 0 ? g.off_cs[0] : g.off_cs[1]) + (je - base);
        const double sj = R.ss[je];
        double dw = 0.0;   // delta_j * omega_j
        if (SCHUR) {
            const double m = R.mm[je];
            double delta;
            if (!TRANS)
                delta = Tb.Gamma * ((dir ? 0.0 : R.gg[je]) * zps - R.gg[je] * zpe + R.ee[je] * zce);
            else
                delta = sj * ((dir ? 0.0 : m) * zps - m * zpe - g.tc * m * zce);
            dw = delta * R.om[je];
        }
        // forward elimination; the register arrays are only indexed by unrolled
        // constants, the last entry is carried separately; all radial values are
        // loaded first (indices clamped to the last point)
        double rv[NRMAX];
#pragma unroll
        for (int q = 0; q < NRMAX; q++) rv[q] = rs[(long long)(q < N ? q : N - 1) * nn];
        // the electrode-level outputs are stored only now, after every load is
        // issued (a load after them would wait for the loads they depend on)
        z[g.off_pe + n] = (TZ)zpe;
        z[g.off_ce + n] = (TZ)zce;
        z[je] = (TZ)zps;
        T y[NRMAX];
        y[0] = (T)(rv[0] * rscale);
        T ylast = y[0];
#pragma unroll
        for (int q = 1; q < NRMAX; q++) {
            if (q < N) {
                const T lq = (T)(TRANS ? Tb.lT[q] : Tb.l[q]);
                y[q] = (T)(rv[q] * rscale) - lq * y[q - 1];
                ylast = y[q];
            }
        }
        T zn = ylast / (T)(Tb.piv[N - 1] + Tb.Gamma * sj);
        zs[(long long)(N - 1) * nn] = (TZ)((double)zn - dw * (TRANS ? Tb.tNT[N - 1] : Tb.tN[N - 1]));
#pragma unroll
        for (int q = NRMAX - 2; q >= 0; q--) {
            if (q < N - 1) {
                const T u = (T)(TRANS ? Tb.tsub[q + 1] : Tb.tsup[q]);
                zn = (y[q] - u * zn) * (T)Tb.ipiv[q];
                zs[(long long)q * nn] = (TZ)((double)zn - dw * (TRANS ? Tb.tNT[q] : Tb.tN[q]));
            }
        }
    };
    // the tables of the node's electrode: through a wave-uniform pointer in the
    // constant address space (scalar loads) when the whole wave lies in one
    // electrode, per lane otherwise
    const int elw = __builtin_amdgcn_readfirstlane(el);
    if (__builtin_amdgcn_ballot_w64(el != elw) == 0) solve(*(const ConstTab *)(R.tabs + elw));
    else solve(R.tabs[el]);
}

// The electrode-level part of z = P^-1 (rscale r): the final level-0
// iterates, identity on the grounded layer
template <typename TZ>
__device__ inline void macro_out_block(const Geom &g, const RadArgs &R, const double *r, double rscale, TZ *z,
                                       int blk)
{
    const long long n = (long long)blk * kBlock + threadIdx.x;
    if (n >= g.nnode) return;
    z[g.off_pe + n] = (TZ)R.x0[2][g.off_pe + n];
    z[g.off_ce + n] = (TZ)R.x0[3][g.off_ce + n];
    const int k = (int)(n / ((long long)g.nx * g.ny));
    const int el = node_mat(g, k);
    if (el < 0) return;
    const long long base = el == 0 ? 0 : g.nea;
    const long long klo = el == 0 ? 0 : g.na + g.ns;
    const long long je = base + n - klo * g.nx * g.ny;
    z[je] = (TZ)(k == 0 ? r[je] * rscale : (el == 0 ? R.x0[0] : R.x0[1])[je]);
}

// The first vector r of a folded cycle at one node: the last two rows of
// A_ss,j^-1 r_s,j (FP64) and the squares of its folded (electrode-level and
// surface) and of its other particle rows
template <int NRMAX, bool TRANS>
__device__ inline void fold_start_node(const Geom &g, const RadialTab *tabs, const double *ss, const double *r,
                                       double *u0, double *u1, long long n, double &sqy, double &sqs)
{
    const int k = (int)(n / ((long long)g.nx * g.ny));
    const double rpe = r[g.off_pe + n], rce = r[g.off_ce + n];
    sqy += rpe * rpe + rce * rce;
    const int el = node_mat(g, k);
    if (el < 0) return;
    const long long base = el == 0 ? 0 : g.nea;
    const long long klo = el == 0 ? 0 : g.na + g.ns;
    const long long je = base + n - klo * g.nx * g.ny;
    const double rps = r[je];
    sqy += rps * rps;
    auto elim = [&](const auto &Tb) {
        const int N = Tb.N;
        const long long nn = el == 0 ? g.nea : g.nec;
        const double *rs = r + (el == 0 ? g.off_cs[0] : g.off_cs[1]) + (je - base);
        double rv[NRMAX];
#pragma unroll
        for (int q = 0; q < NRMAX; q++) rv[q] = rs[(long long)(q < N ? q : N - 1) * nn];
        double y = rv[0], ym = 0.0;
        double sq = rv[0] * rv[0], rl = rv[0];
#pragma unroll
        for (int q = 1; q < NRMAX; q++) {
            if (q < N) {
                ym = y;
                y = rv[q] - (TRANS ? Tb.lT[q] : Tb.l[q]) * y;
                rl = rv[q];
                if (q < N - 1) sq += rv[q] * rv[q];
            }
        }
        sqs += sq;
        sqy += rl * rl;
        const double zn = y / (Tb.piv[N - 1] + Tb.Gamma * ss[je]);
        u0[je] = zn;
        u1[je] = (ym - (TRANS ? Tb.tsub[N - 1] : Tb.tsup[N - 2]) * zn) * Tb.ipiv[N - 2];
    };
    const int elw = __builtin_amdgcn_readfirstlane(el);
    if (__builtin_amdgcn_ballot_w64(el != elw) == 0) elim(*(const ConstTab *)(tabs + elw));
    else elim(tabs[el]);
}

// The update x (+)= sum_k y_k z_k of a folded cycle at one node: the
// electrode-level rows from the stored directions; the particle rows of each
// direction from those and A_ss^-1 s (s: the particle rows of the cycle's first
// vector, solved once), rounded and added up one direction after the other
// like stored ones.  (Summed before the solve, the particle surface rows carry
// a third of the rounding, which is the largest part of the true residual: such
// solves stop now and then a cycle earlier than those with whole vectors.)
struct FoldUpdate {
    const RadialTab *tabs;
    const double *gg, *ss, *ee, *mm, *om;
    const double *v0, *V, *Z, *y, *alpha, *invbeta;   // V_q (q >= 1) at V + q (Nm + ne)
    double *x;
    int nv, add;
};
template <int NRMAX, bool TRANS>
__device__ inline void fold_update_node(const Geom &g, const FoldUpdate &U, long long n)
{
    const int k = (int)(n / ((long long)g.nx * g.ny));
    const int el = node_mat(g, k);
    const long long base = el == 0 ? 0 : g.nea;
    const long long klo = el == 0 ? 0 : g.na + g.ns;
    const long long je = base + n - klo * g.nx * g.ny;   // (electrode nodes)
    const long long pe = g.off_pe + n, ce = g.off_ce + n, ld = g.Nm;
    double xpe = U.add ? U.x[pe] : 0.0, xce = U.add ? U.x[ce] : 0.0;
    if (el < 0) {
        for (int q = 0; q < U.nv; q++) {
            xpe += U.y[q] * U.Z[q * ld + pe];
            xce += U.y[q] * U.Z[q * ld + ce];
        }
        U.x[pe] = xpe;
        U.x[ce] = xce;
        return;
    }
    const bool dir = (k == 0);
    auto solve = [&](const auto &Tb) {
        const int N = Tb.N;
        const long long nn = el == 0 ? g.nea : g.nec;
        const long long offs = (el == 0 ? g.off_cs[0] : g.off_cs[1]) + (je - base);
        const double *rs = U.v0 + offs;
        double *xs = U.x + offs;
        const double sj = U.ss[je], m = U.mm[je], gj = U.gg[je], ej = U.ee[je], om = U.om[je];
        // u = A_ss^-1 s, in place over the column
        double u[NRMAX], xv[NRMAX];
#pragma unroll
        for (int q = 0; q < NRMAX; q++) u[q] = rs[(long long)(q < N ? q : N - 1) * nn];
        if (U.add) {
#pragma unroll
            for (int q = 0; q < NRMAX; q++) xv[q] = xs[(long long)(q < N ? q : N - 1) * nn];
        } else {
#pragma unroll
            for (int q = 0; q < NRMAX; q++) xv[q] = 0.0;
        }
        double xps = U.add ? U.x[je] : 0.0;
        const double sN = U.v0[fold_at(fold_map(g), g.Nm + je)];
        double ul = u[0];
#pragma unroll
        for (int q = 1; q < NRMAX; q++) {
            if (q < N) {
                u[q] -= (TRANS ? Tb.lT[q] : Tb.l[q]) * u[q - 1];
                ul = u[q];
            }
        }
        double zn = ul / (Tb.piv[N - 1] + Tb.Gamma * sj);
#pragma unroll
        for (int q = NRMAX - 1; q >= 0; q--) {
            if (q == N - 1) u[q] = zn;
            if (q < N - 1) {
                zn = (u[q] - (TRANS ? Tb.tsub[q + 1 < kMaxNr ? q + 1 : q] : Tb.tsup[q]) * zn) * Tb.ipiv[q];
                u[q] = zn;
            }
        }
        for (int p = 0; p < U.nv; p++) {
            const double zps = U.Z[p * ld + je], zpe = U.Z[p * ld + pe], zce = U.Z[p * ld + ce];
            const double sc = U.invbeta[p], yp = U.y[p], ap = U.alpha[p] * sc;
            const double e = p > 0 ? U.V[p * (ld + g.ne) + ld + je] * sc - ap * sN : 0.0;
            const double dw = fold_delta<TRANS>(g, Tb, dir, m, gj, sj, ej, zps, zpe, zce) * om, eo = e * om;
            xps += yp * zps;
            xpe += yp * zpe;
            xce += yp * zce;
#pragma unroll
            for (int q = 0; q < NRMAX; q++) {
                if (q < N) {
                    xv[q] += yp * fold_row(ap, u[q], eo, dw, TRANS ? Tb.tNT[q] : Tb.tN[q]);
                }
            }
        }
        U.x[je] = xps;
        U.x[pe] = xpe;
        U.x[ce] = xce;
#pragma unroll
        for (int q = 0; q < NRMAX; q++)
            if (q < N) xs[(long long)q * nn] = xv[q];
    };
    // the electrode's table through a wave-uniform pointer (scalar loads) when
    // the whole wave lies in one electrode, per lane otherwise
    const int elw = __builtin_amdgcn_readfirstlane(el);
    if (__builtin_amdgcn_ballot_w64(el != elw) == 0) solve(*(const ConstTab *)(U.tabs + elw));
    else solve(U.tabs[el]);
}

// ---------------------------------------------------------------------------
// The operator y = A x (or A^T x, or b - A x) for the nodes of one block,
// with the sum of squares of what the thread writes (paper Sec. 4.1,
// eq. blocks; see operator.hip).
// ---------------------------------------------------------------------------
struct OpArgs {
    const RadialTab *tabs;
    const double *sigh, *kaph, *gg, *ss, *ee, *mm;
    const void *x;       // TX
    double *y;
    const double *b;     // b - A x when not null
    const double *om;    // omega per electrode node (Schur complement operator)
    const double *kdh;   // h * diffusion-potential coefficient per element (GEN)
    const double *dch;   // h * c_e diffusion coefficient per element (GEN)
    FoldVec fv;          // OP_FOLD
};

// Forms of the operator: A on whole vectors; the Schur complement of the
// particle blocks on electrode-level vectors (the reaction scaled by omega_j,
// no particle column); A on the direction of a folded vector, of which x holds
// the electrode-level rows (the surface rows of y after its electrode-level
// ones)
enum OpMode { OP_FULL = 0, OP_RED = 1, OP_FOLD = 2 };

// the last two rows of the particle column of a folded vector's direction
template <bool TRANS, typename Tab>
__device__ inline void fold_surface(const Geom &g, const OpArgs &O, const Tab &T, long long je, bool dir, double m,
                                    double gj, double sj, double ej, double zps, double zpe, double zce, double &xsN,
                                    double &xsM)
{
    const int N = T.N;
    const FoldNode fn = fold_node(g, O.fv, je);
    const double om = O.om[je];
    const double dw = fold_delta<TRANS>(g, T, dir, m, gj, sj, ej, zps, zpe, zce) * om, eo = fn.e * om;
    xsN = fold_row(fn.ap, O.fv.u0[je], eo, dw, TRANS ? T.tNT[N - 1] : T.tN[N - 1]);
    xsM = fold_row(fn.ap, O.fv.u1[je], eo, dw, TRANS ? T.tNT[N - 2] : T.tN[N - 2]);
}

template <typename TX>
__device__ inline double ldx(const TX *p) { return (double)*p; }

// The node's neighbourhood in f, absent neighbours as zeros.  An absent
// neighbour's index is clamped to the node and its value dropped by a select,
// so that the loads are in flight together (bounds tests around them became
// branches, with one wait per load).
template <typename TX>
__device__ inline void load_nb(const Geom &g, const TX *f, long long n, const NbMask &M, double X[27])
{
    const TX *fn = f + n;
#pragma unroll
    for (int o = 0; o < 27; o++)
        X[o] = ldx(fn + (((o % 3 - 1) + g.nx * ((o / 3) % 3 - 1 + g.ny * (o / 9 - 1))) & -M.has(o)));
#pragma unroll
    for (int o = 0; o < 27; o++) X[o] = M.has(o) ? X[o] : 0.0;
}

// The eight elements of a node (e = ex + 2 ey + 4 ez, ex: the upper one along
// x), absent ones clamped to one that is there
struct NodeElems {
    unsigned x, y, z;
    int ix[2], iy[2], iz[2];
    __device__ NodeElems(const Geom &g, int i, int j, int k)
        : x((i > 0 ? 1u : 0u) | (i < g.nx - 1 ? 2u : 0u)), y((j > 0 ? 1u : 0u) | (j < g.ny - 1 ? 2u : 0u)),
          z((k > 0 ? 1u : 0u) | (k < g.nz - 1 ? 2u : 0u))
    {
        ix[0] = i > 0 ? i - 1 : 0;
        ix[1] = i < g.nx - 1 ? i : i - 1;
        iy[0] = (g.nx - 1) * (j > 0 ? j - 1 : 0);
        iy[1] = (g.nx - 1) * (j < g.ny - 1 ? j : j - 1);
        iz[0] = (g.nx - 1) * (g.ny - 1) * (k > 0 ? k - 1 : 0);
        iz[1] = (g.nx - 1) * (g.ny - 1) * (k < g.nz - 1 ? k : k - 1);
    }
    __device__ int has(int e) const { return (x >> (e & 1)) & (y >> ((e >> 1) & 1)) & (z >> (e >> 2)) & 1u; }
    __device__ int id(int e) const { return ix[e & 1] + iy[(e >> 1) & 1] + iz[e >> 2]; }
    __device__ void load(const double *C, double c[8]) const
    {
#pragma unroll
        for (int e = 0; e < 8; e++) c[e] = C[id(e)];
#pragma unroll
        for (int e = 0; e < 8; e++) c[e] = has(e) ? c[e] : 0.0;
    }
};

// Stencil parts of the operator at one node, gathered either per node from
// memory or from an LDS tile: K_kappa phi_e, K_kappa c_e, M_eps c_e and, on
// electrode nodes, K_sigma phi_s, with the centre values (xpsc is phi_s as a
// neighbour value: zero on the grounded layer).
struct OpStencil {
    double Kpe, xpe, Kce, Mce, xce, Kps, xpsc;
    double Kx;   // GEN: the diffusion-potential stiffness applied to c_e (phi_e if transposed)
    double Npe = 0.0, Nce = 0.0;   // GEN: Newton terms of the phi_e and c_e rows
};

// Newton terms at one node (GEN, g.nwu set): each element e of the node
// has coefficients that depend on its mean c_e, so it adds to its corner
// rows (K_e u)_a times the mean of x_ce over its corners, with K_e the
// element stiffness (over h) and u the state: phi_e rows da_e (K_e phi_e) +
// db_e (K_e c_e), c_e rows dc_e (K_e c_e).  Transposed, the node (a c_e
// column) collects w_e^T (...) / 8 from each of its elements, w the input's
// phi_e and c_e on the element's corners.  Xc: the input's c_e around the
// node (the forward form).  (K_e u)_a = sum_{b != a} kw[a^b] (u_a - u_b).
template <typename TX, bool TRANS>
__device__ inline void newton_terms(const Geom &g, const TX *x, long long n, int i, int j, int k, const NbMask &M,
                                    const NodeElems &E, const double Xc[27], OpStencil &P)
{
    const double *up = g.nwu + g.off_pe, *uc = g.nwu + g.off_ce;
    double npe = 0.0, nce = 0.0;
    if (!TRANS) {
        // one 27-value neighbourhood at a time: the means of x_ce, then the
        // sums over the state's phi_e, then those over its c_e.  An absent
        // element's coefficients are zeros, and so are its terms.
        double xm[8], sp[8], sc[8], U[27];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            xm[e] = 0.0;
#pragma unroll
            for (int b = 0; b < 8; b++)
                xm[e] += Xc[nb_index((e & 1) - 1 + (b & 1), ((e >> 1) & 1) - 1 + ((b >> 1) & 1), (e >> 2) - 1 + (b >> 2))];
            xm[e] *= 0.125;
        }
        auto sums = [&](double s[8]) {
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const int a = e ^ 7;   // this node's corner of the element
                s[e] = 0.0;
#pragma unroll
                for (int b = 0; b < 8; b++)
                    if (b != a)
                        s[e] += g.kw[a ^ b] * (U[13] - U[nb_index((e & 1) - 1 + (b & 1), ((e >> 1) & 1) - 1 + ((b >> 1) & 1),
                                                                  (e >> 2) - 1 + (b >> 2))]);
            }
        };
        // (finished before the next loads, as in operator_node)
        auto done = [](double v[8]) {
            __asm__ volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]),
                             "+v"(v[7]) : : "memory");
        };
        done(xm);
        load_nb(g, up, n, M, U);
        sums(sp);
        done(sp);
        load_nb(g, uc, n, M, U);
        sums(sc);
        done(sc);
        double A[8], B[8], C[8];
        E.load(g.nwa, A);
        E.load(g.nwb, B);
        E.load(g.nwc, C);
#pragma unroll
        for (int e = 0; e < 8; e++) {
            npe += (A[e] * sp[e] + B[e] * sc[e]) * xm[e];
            nce += C[e] * sc[e] * xm[e];
        }
    } else {
        const long long layer = (long long)g.nx * g.ny;
        for (int e = 0; e < 8; e++) {
            // (the element from the node again: E indexed by a variable leaves the
            // registers, in the whole kernel; the transposed operator, also
            // without these terms, then took 79 us for 54 over the electrode-level
            // unknowns of 64 x 64 x 192 nodes)
            const int ei = i - 1 + (e & 1), ej = j - 1 + ((e >> 1) & 1), ek = k - 1 + (e >> 2);
            if (ei < 0 || ej < 0 || ek < 0 || ei >= g.nx - 1 || ej >= g.ny - 1 || ek >= g.nz - 1) continue;
            const int id = ei + (g.nx - 1) * (ej + (g.ny - 1) * ek);
            const double A = g.nwa[id], B = g.nwb[id], C = g.nwc[id];
            // corner b of the element
            const long long c0 = ei + (long long)g.nx * ej + layer * ek;
            auto node = [&](int b) { return c0 + (b & 1) + (long long)g.nx * ((b >> 1) & 1) + layer * ((b >> 2) & 1); };
            double t = 0.0;
            for (int a = 0; a < 8; a++) {
                const long long na = node(a);
                double kup = 0.0, kuc = 0.0;
                for (int b = 0; b < 8; b++) {
                    if (b == a) continue;
                    const long long nb = node(b);
                    const double w = g.kw[a ^ b];
                    kup += w * (up[na] - up[nb]);
                    kuc += w * (uc[na] - uc[nb]);
                }
                t += ldx(x + g.off_pe + na) * (A * kup + B * kuc) + ldx(x + g.off_ce + na) * C * kuc;
            }
            nce += 0.125 * t;
        }
    }
    P.Npe = npe;
    P.Nce = nce;
}

// Reaction coupling of one electrode node: the linearized reaction q and the
// weights with which it enters the phi_s, phi_e, c_e and surface c_s rows
// (a = (m, -m, -tc m, Gamma), b = (g, -g, e, s); transposed: a and b swap).
struct OpCoupling {
    double q, r0, r1, r2, r3;
};
template <bool TRANS, typename Tab>
__device__ inline OpCoupling op_coupling(const Geom &g, const Tab &T, bool dir, double m,
                                         double gj, double sj, double ej, double xpsc, double xpe,
                                         double xce, double xsN)
{
    OpCoupling c;
    const double a0 = dir ? 0.0 : m, b0 = dir ? 0.0 : gj;
    if (!TRANS) {
        c.q = b0 * xpsc - gj * xpe + ej * xce + sj * xsN;
        c.r0 = a0; c.r1 = -m; c.r2 = -g.tc * m; c.r3 = T.Gamma;
    } else {
        c.q = a0 * xpsc - m * xpe - g.tc * m * xce + T.Gamma * xsN;
        c.r0 = b0; c.r1 = -gj; c.r2 = ej; c.r3 = sj;
    }
    return c;
}

// Row r of T0 (or T0^T) applied to a particle column, without the coupling
template <typename Tab>
__device__ inline double op_radial_row(const Tab &T, bool trans, int r, int N, double xm, double x0,
                                       double xp)
{
    if (!trans) return T.tdia[r] * x0 + T.tsub[r] * xm + T.tsup[r] * xp;
    return T.tdia[r] * x0 + (r > 0 ? T.tsup[r > 0 ? r - 1 : 0] : 0.0) * xm +
           (r < N - 1 ? T.tsub[r + 1 < kMaxNr ? r + 1 : r] : 0.0) * xp;
}

// Everything after the stencil parts: reaction coupling, radial rows and
// the output (y, or b - A x when RESID); returns the sum of squares written.
// GEN: separate element coefficients for the diffusion-potential block
// (P.Kx) and the c_e diffusion (P.Kce), instead of chi * kappa and kappa.
// MODE: see OpMode
template <typename TX, int NRMAX, bool TRANS, bool RESID, bool GEN = false, int MODE = OP_FULL>
__device__ inline double operator_finish(const Geom &g, const OpArgs &O, long long n, int i, int j,
                                         int k, const OpStencil &P)
{
    const TX *x = (const TX *)O.x;
    double *y = O.y;
    const double *b = O.b;
    double sq = 0.0;
    const double xpe = P.xpe, xce = P.xce;
    // b - A x: every value of b this node needs is loaded before its first
    // store (a load after a store may not be hoisted above it, pointers may
    // alias, and would wait for the loads the stored value depends on)
    double bpe = 0.0, bce = 0.0;
    if (RESID) {
        bpe = b[g.off_pe + n];
        bce = b[g.off_ce + n];
    }
    double ype, yce;
    if (GEN) {
        ype = (TRANS ? P.Kpe : P.Kpe + P.Kx) + P.Npe;
        yce = (TRANS ? P.Mce + P.Kce + P.Kx : P.Mce + P.Kce) + P.Nce;
    } else if (!TRANS) {
        ype = P.Kpe + g.chi * P.Kce;
        yce = P.Mce + P.Kce;
    } else {
        ype = P.Kpe;
        yce = P.Mce + P.Kce + g.chi * P.Kpe;
    }
    const int el = node_mat(g, k);
    if (el >= 0) {
        const long long base = el == 0 ? 0 : g.nea;
        const int klo = el == 0 ? 0 : g.na + g.ns;
        const long long je = base + i + (long long)g.nx * (j + (long long)g.ny * (k - klo));
        const bool dir = (k == 0);
        const double xps = ldx(x + je);
        auto rows = [&](const auto &T) {
            const int N = T.N;
            const long long nn = el == 0 ? g.nea : g.nec;
            const long long jl = je - base;
            const long long offs = el == 0 ? g.off_cs[0] : g.off_cs[1];
            const TX *xs = x + offs + jl;
            double *ys = y + offs + jl;
            const double m = O.mm[je], gj = O.gg[je], sj = O.ss[je], ej = O.ee[je];
            // the particle column, loaded at once (indices clamped to the last point)
            double xr[NRMAX], bv[NRMAX];
            double xsN = 0.0, xsM = 0.0, bps = 0.0;
            if (MODE == OP_FOLD) fold_surface<TRANS>(g, O, T, je, dir, m, gj, sj, ej, P.xpsc, xpe, xce, xsN, xsM);
            if (MODE == OP_FULL) {
#pragma unroll
                for (int r = 0; r < NRMAX; r++) xr[r] = ldx(xs + (long long)(r < N ? r : N - 1) * nn);
                if (RESID) {
#pragma unroll
                    for (int r = 0; r < NRMAX; r++) bv[r] = b[offs + jl + (long long)(r < N ? r : N - 1) * nn];
                }
                xsN = xr[0];
#pragma unroll
                for (int r = 1; r < NRMAX; r++)
                    if (r == N - 1) xsN = xr[r];
            }
            if (RESID) bps = b[je];
            const OpCoupling cp = op_coupling<TRANS>(g, T, dir, m, gj, sj, ej, P.xpsc, xpe, xce, xsN);
            const double q = MODE == OP_RED ? cp.q * O.om[je] : cp.q, r3 = cp.r3;
            double yps = dir ? xps : P.Kps + cp.r0 * q;
            ype += cp.r1 * q;
            yce += cp.r2 * q;
            if (RESID) yps = bps - yps;
            y[je] = yps;
            sq += yps * yps;
            if (MODE == OP_FOLD) y[g.Nm + je] = op_radial_row(T, TRANS, N - 1, N, xsM, xsN, 0.0) + r3 * q;
#pragma unroll
            for (int r = 0; r < NRMAX; r++) {
                if (MODE != OP_FULL) break;
                if (r < N) {
                    const double xm = r > 0 ? xr[r > 0 ? r - 1 : 0] : 0.0;
                    const double x0 = xr[r];
                    const double xp = r < N - 1 ? xr[r + 1 < NRMAX ? r + 1 : r] : 0.0;
                    double v = op_radial_row(T, TRANS, r, N, xm, x0, xp);
                    if (r == N - 1) v += r3 * q;
                    if (RESID) v = bv[r] - v;
                    ys[(long long)r * nn] = v;
                    sq += v * v;
                }
            }
        };
        // the electrode's table through a wave-uniform pointer (scalar loads)
        // when the whole wave lies in one electrode, per lane otherwise
        const int elw = __builtin_amdgcn_readfirstlane(el);
        if (__builtin_amdgcn_ballot_w64(el != elw) == 0) rows(*(const ConstTab *)(O.tabs + elw));
        else rows(O.tabs[el]);
    }
    if (RESID) {
        ype = bpe - ype;
        yce = bce - yce;
    }
    y[g.off_pe + n] = ype;
    y[g.off_ce + n] = yce;
    sq += ype * ype + yce * yce;
    return sq;
}

// The operator y = A x (or A^T x, or b - A x) at one node, every stencil
// value read from memory (paper Sec. 4.1, eq. blocks; see operator.hip).
template <typename TX, int NRMAX, bool TRANS, bool RESID, bool GEN = false, int MODE = OP_FULL>
__device__ inline double operator_node(const Geom &g, const OpArgs &O, long long n)
{
    const TX *x = (const TX *)O.x;
    const int i = (int)(n % g.nx);
    const long long t = n / g.nx;
    const int j = (int)(t % g.ny), k = (int)(t / g.ny);
    const NbMask M(i, j, k, g.nx, g.ny, g.nz);
    const NodeElems E(g, i, j, k);
    // element coefficients of the node's eight elements; each set is read
    // beside the neighbourhood that uses it, so only one set is live at a time
    double ck[8], cs[8], cm[8];
    E.load(O.kaph, ck);
    OpStencil P;
    double X[27];
    P.Kx = 0.0;
    load_nb(g, x + g.off_pe, n, M, X);
    P.Kpe = stiff_of<GEN>(g, ck, X);
    P.xpe = X[13];
    if (GEN && TRANS) {
        double cx[8];
        E.load(O.kdh, cx);
        P.Kx = stiff_of<GEN>(g, cx, X);
    }
    // an empty statement that takes the finished sums: they may not be
    // deferred past it nor the next neighbourhood's loads hoisted above it,
    // so one 27-value neighbourhood is live at a time (register use)
    __asm__ volatile("" : "+v"(P.Kpe), "+v"(P.Kx) : : "memory");
    load_nb(g, x + g.off_ce, n, M, X);
    if (GEN) {
        double cd[8], cx[8];
        E.load(O.dch, cd);
        P.Kce = stiff_of<GEN>(g, cd, X);
        if (!TRANS) {
            E.load(O.kdh, cx);
            P.Kx = stiff_of<GEN>(g, cx, X);
        }
    } else {
        P.Kce = stiff_of<GEN>(g, ck, X);
    }
    // per-element storage only with separate coefficients (GEN)
    if (GEN && g.meh) {
        E.load((const double *)(const __attribute__((address_space(1))) double *)g.meh, cm);
    } else {
#pragma unroll
        for (int e = 0; e < 8; e++)
            cm[e] = E.has(e) ? (elem_mat(g, k - 1 + (e >> 2)) >= 0 ? g.mass_elec : g.mass_sep) : 0.0;
    }
    P.Mce = q1_mass(cm, X);
    P.xce = X[13];
    if (GEN) __asm__ volatile("" : "+v"(P.Kce), "+v"(P.Mce), "+v"(P.Kx) : : "memory");
    if (GEN && g.nwu) newton_terms<TX, TRANS>(g, x, n, i, j, k, M, E, X, P);
    __asm__ volatile("" : "+v"(P.Kce), "+v"(P.Mce), "+v"(P.Kx), "+v"(P.Npe), "+v"(P.Nce) : : "memory");
    P.Kps = 0.0;
    P.xpsc = 0.0;
    const int el = node_mat(g, k);
    if (el >= 0) {
        E.load(O.sigh, cs);
        const long long base = el == 0 ? 0 : g.nea;
        const int klo = el == 0 ? 0 : g.na + g.ns;
        const int khi = el == 0 ? g.na - 1 : g.nz - 1;
        const long long je = base + i + (long long)g.nx * (j + (long long)g.ny * (k - klo));
        // phi_s neighbours: same electrode, grounded layer as a zero column
        NbMask S = M;
        S.z = (k > klo && k != 1 ? 1u : 0u) | (k != 0 ? 2u : 0u) | (k < khi ? 4u : 0u);
        load_nb(g, x, je, S, X);
        P.Kps = stiff_of<GEN>(g, cs, X);
        P.xpsc = X[13];
    }
    return operator_finish<TX, NRMAX, TRANS, RESID, GEN, MODE>(g, O, n, i, j, k, P);
}

// ---------------------------------------------------------------------------
// The operator over a 2.5D tile (the level-0 smoother's scheme): a TX x TY
// block of nodes marches through CZ node layers; three planes of phi_e, c_e
// and phi_s with a one-node halo and two layers of element coefficients sit
// in LDS rings, fetched into registers one layer ahead.  Each node's
// arithmetic is operator_finish on the same stencil values as operator_node,
// so both give the same result.
// ---------------------------------------------------------------------------
struct OpLds {
    double pe[3][kXpLds], ce[3][kXpLds], ps[3][kXpLds];
    double kap[2][kCkLds], sig[2][kCkLds];
};

__host__ __device__ inline int op_tiles(int nx, int ny, int nz, int TX, int CZ)
{
    return smooth0_box_tiles(nx, ny, nz, TX, CZ);
}

// MODE: see OpMode (OP_RED: 1 - Gamma s_j (A_ss,j^-1)_NN = omega_j by
// Sherman-Morrison)
template <typename TX_T, bool TRANS, int MODE = OP_FULL>
__device__ inline void operator_tile(const Geom &g, const OpArgs &O, double *qout, int tile, int TX,
                                     int CZ, OpLds &L)
{
    const TX_T *x = (const TX_T *)O.x;
    const int TY = kBlock / TX;
    const int PX = TX + 2, PY = TY + 2;
    const int EX = TX + 1, EY = TY + 1;
    const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY;
    const int tix = tile % ntx, tiy = (tile / ntx) % nty, tch = tile / (ntx * nty);
    const int i0 = tix * TX, j0 = tiy * TY, k0 = tch * CZ;
    const int k1 = k0 + CZ < g.nz ? k0 + CZ : g.nz;
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    const int i = i0 + tx, j = j0 + ty;
    const bool own = i < g.nx && j < g.ny;
    const long long layer = (long long)g.nx * g.ny;

    double pe[2], ce[2], ps[2], kp[2], sg[2];
    auto fetch_planes_to = [&](int kk, double vpe[2], double vce[2], double vps[2]) {
        const int el = (kk >= 0 && kk < g.nz) ? node_mat(g, kk) : -1;
        const bool has_ps = el >= 0 && kk != 0;
        const long long psb = el == 0 ? 0 : g.nea - (long long)(g.na + g.ns) * layer;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            const int ii = i0 - 1 + q % PX, jj = j0 - 1 + q / PX;
            const bool ok = q < PX * PY && kk >= 0 && kk < g.nz && ii >= 0 && ii < g.nx && jj >= 0 &&
                            jj < g.ny;
            const long long nd = ii + g.nx * (jj + (long long)g.ny * kk);
            vpe[h] = ok ? ldx(x + g.off_pe + nd) : 0.0;
            vce[h] = ok ? ldx(x + g.off_ce + nd) : 0.0;
            vps[h] = (ok && has_ps) ? ldx(x + (psb + nd)) : 0.0;
        }
    };
    auto store_planes_from = [&](int slot, const double vpe[2], const double vce[2], const double vps[2]) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            if (q < PX * PY) {
                L.pe[slot][q] = vpe[h];
                L.ce[slot][q] = vce[h];
                L.ps[slot][q] = vps[h];
            }
        }
    };
    auto fetch_elems_to = [&](int ek, double vkp[2], double vsg[2]) {
        const bool lay = ek >= 0 && ek < g.nz - 1;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            const int ei = i0 - 1 + q % EX, ej = j0 - 1 + q / EX;
            const bool ok = q < EX * EY && lay && ei >= 0 && ei < g.nx - 1 && ej >= 0 && ej < g.ny - 1;
            const long long id = ei + (long long)(g.nx - 1) * (ej + (long long)(g.ny - 1) * ek);
            vkp[h] = ok ? O.kaph[id] : 0.0;
            vsg[h] = ok ? O.sigh[id] : 0.0;
        }
    };
    auto store_elems_from = [&](int slot, const double vkp[2], const double vsg[2]) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = threadIdx.x + h * kBlock;
            if (q < EX * EY) {
                L.kap[slot][q] = vkp[h];
                L.sig[slot][q] = vsg[h];
            }
        }
    };
    auto fetch_planes = [&](int kk) { fetch_planes_to(kk, pe, ce, ps); };
    auto store_planes = [&](int slot) { store_planes_from(slot, pe, ce, ps); };
    auto fetch_elems = [&](int ek) { fetch_elems_to(ek, kp, sg); };
    auto store_elems = [&](int slot) { store_elems_from(slot, kp, sg); };
    {   // prologue: every load of the first layer is issued before any of
        // them is stored, so the tile waits for one memory latency, not four
        double pe0[2], ce0[2], ps0[2], pe1[2], ce1[2], ps1[2], kp0[2], sg0[2];
        fetch_planes_to(k0 - 1, pe0, ce0, ps0);
        fetch_planes_to(k0, pe1, ce1, ps1);
        fetch_elems_to(k0 - 1, kp0, sg0);
        fetch_planes(k0 + 1);
        fetch_elems(k0);
        store_planes_from((k0 + 2) % 3, pe0, ce0, ps0);
        store_planes_from(k0 % 3, pe1, ce1, ps1);
        store_elems_from((k0 + 1) & 1, kp0, sg0);
    }
    for (int k = k0; k < k1; k++) {
        store_planes((k + 1) % 3);
        store_elems(k & 1);
        __syncthreads();
        if (k + 1 < k1) {
            fetch_planes(k + 2);
            fetch_elems(k + 1);
        }
        if (own) {
            // element coefficients are read from LDS (or formed) just before
            // the field that uses them, so only one set is live at a time
            auto elem_coef = [&](const double (*C)[kCkLds], double c[8]) {
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const int ex = e & 1, ey = (e >> 1) & 1, ez = (e >> 2) & 1;
                    c[e] = C[(k - 1 + ez) & 1][(tx + ex) + EX * (ty + ey)];
                }
            };
            auto mass_coef = [&](double c[8]) {
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const int ex = e & 1, ey = (e >> 1) & 1, ez = (e >> 2) & 1;
                    const int ek = k - 1 + ez;
                    // the element exists iff its kappa coefficient slot was
                    // filled; decide by the indices, as the per-node gather does
                    const int ei = i - 1 + ex, ej = j - 1 + ey;
                    const bool ok = ei >= 0 && ej >= 0 && ek >= 0 && ei < g.nx - 1 && ej < g.ny - 1 &&
                                    ek < g.nz - 1;
                    c[e] = ok ? (elem_mat(g, ek) >= 0 ? g.mass_elec : g.mass_sep) : 0.0;
                }
            };
            double ck[8], cs[8], cm[8];
            elem_coef(L.kap, ck);
            OpStencil P;
            double X[27];
            auto gather = [&](const double (*F)[kXpLds]) {
#pragma unroll
                for (int dz = -1; dz <= 1; dz++) {
                    const double *Pl = F[(k + dz + 3) % 3];
#pragma unroll
                    for (int dy = -1; dy <= 1; dy++)
#pragma unroll
                        for (int dx = -1; dx <= 1; dx++)
                            X[nb_index(dx, dy, dz)] = Pl[(tx + 1 + dx) + PX * (ty + 1 + dy)];
                }
            };
            // one field at a time: the scheduling barriers keep the three
            // 27-value gathers from being hoisted together (register use)
            gather(L.pe);
            P.Kpe = q1_stiff(ck, X);
            P.xpe = X[13];
            // an empty statement that takes the finished sum: the compiler
            // may neither defer the sum nor hoist the next gather above it,
            // so only one 27-value neighbourhood is live at a time
            __asm__ volatile("" : "+v"(P.Kpe) : : "memory");
            gather(L.ce);
            P.Kce = q1_stiff(ck, X);
            mass_coef(cm);
            P.Mce = q1_mass(cm, X);
            P.xce = X[13];
            __asm__ volatile("" : "+v"(P.Kce), "+v"(P.Mce) : : "memory");
            P.Kps = 0.0;
            P.xpsc = 0.0;
            if (node_mat(g, k) >= 0) {
                elem_coef(L.sig, cs);
                gather(L.ps);
                P.Kps = q1_stiff(cs, X);
                P.xpsc = X[13];
            }
            const long long n = i + (long long)g.nx * j + layer * k;
            double ype, yce;
            if (!TRANS) {
                ype = P.Kpe + g.chi * P.Kce;
                yce = P.Mce + P.Kce;
            } else {
                ype = P.Kpe;
                yce = P.Mce + P.Kce + g.chi * P.Kpe;
            }
            const int el = node_mat(g, k);
            if (el >= 0) {
                const long long base = el == 0 ? 0 : g.nea;
                const int klo = el == 0 ? 0 : g.na + g.ns;
                const long long je = base + i + (long long)g.nx * (j + (long long)g.ny * (k - klo));
                const bool dir = (k == 0);
                // the tile's layer lies in one electrode: its table through a
                // wave-uniform pointer (scalar loads)
                const ConstTab &T = *(const ConstTab *)(O.tabs + __builtin_amdgcn_readfirstlane(el));
                double xsN = 0.0, xsM = 0.0;
                const double m = O.mm[je], gj = O.gg[je], sj = O.ss[je], ej = O.ee[je];
                if (MODE == OP_FULL) {
                    const long long nn = el == 0 ? g.nea : g.nec;
                    const long long offs = el == 0 ? g.off_cs[0] : g.off_cs[1];
                    xsN = ldx(x + offs + (je - base) + (long long)(T.N - 1) * nn);
                }
                if (MODE == OP_FOLD)
                    fold_surface<TRANS>(g, O, T, je, dir, m, gj, sj, ej, P.xpsc, P.xpe, P.xce, xsN, xsM);
                const OpCoupling cp = op_coupling<TRANS>(g, T, dir, m, gj, sj, ej, P.xpsc, P.xpe, P.xce, xsN);
                const double q = MODE == OP_RED ? cp.q * O.om[je] : cp.q;
                O.y[je] = dir ? ldx(x + je) : P.Kps + cp.r0 * q;
                ype += cp.r1 * q;
                yce += cp.r2 * q;
                if (MODE == OP_FULL) qout[je] = q;
                if (MODE == OP_FOLD)
                    O.y[g.Nm + je] = op_radial_row(T, TRANS, T.N - 1, T.N, xsM, xsN, 0.0) + cp.r3 * q;
            }
            O.y[g.off_pe + n] = ype;
            O.y[g.off_ce + n] = yce;
        }
        __syncthreads();
    }
}


// The particle rows of y = A x (or A^T x) for one electrode node je: row r
// of T0 applied to its column (loaded at once, indices clamped to the last
// point), plus the coupling weight times q (stored by operator_tile) on the
// surface row.
template <typename TX_T, int NRMAX, bool TRANS>
__device__ inline void operator_radial(const Geom &g, const OpArgs &O, const double *q, long long je)
{
    const TX_T *x = (const TX_T *)O.x;
    const int el = je < g.nea ? 0 : 1;
    const long long nn = el == 0 ? g.nea : g.nec;
    const long long jl = el == 0 ? je : je - g.nea;
    const long long offs = el == 0 ? g.off_cs[0] : g.off_cs[1];
    const TX_T *xs = x + offs + jl;
    double *ys = O.y + offs + jl;
    auto rows = [&](const auto &T) {
        const int N = T.N;
        double xr[NRMAX];
#pragma unroll
        for (int r = 0; r < NRMAX; r++) xr[r] = ldx(xs + (long long)(r < N ? r : N - 1) * nn);
        const double r3 = TRANS ? O.ss[je] : T.Gamma, qj = q[je];
        // all rows first, then the stores: a table read after a store may not
        // be hoisted above it (the pointers may alias), which would chain the
        // rows' cache latencies
        double v[NRMAX];
#pragma unroll
        for (int r = 0; r < NRMAX; r++) {
            if (r < N) {
                const double xm = r > 0 ? xr[r > 0 ? r - 1 : 0] : 0.0;
                const double xp = r < N - 1 ? xr[r + 1 < NRMAX ? r + 1 : r] : 0.0;
                v[r] = op_radial_row(T, TRANS, r, N, xm, xr[r], xp);
                if (r == N - 1) v[r] += r3 * qj;   // the same expression as in operator_finish
            }
        }
#pragma unroll
        for (int r = 0; r < NRMAX; r++)
            if (r < N) ys[(long long)r * nn] = v[r];
    };
    // the electrode's table through a wave-uniform pointer (scalar loads) when
    // the whole wave lies in one electrode, per lane otherwise
    const int elw = __builtin_amdgcn_readfirstlane(el);
    if (__builtin_amdgcn_ballot_w64(el != elw) == 0) rows(*(const ConstTab *)(O.tabs + elw));
    else rows(O.tabs[el]);
}

}  // namespace p4d
