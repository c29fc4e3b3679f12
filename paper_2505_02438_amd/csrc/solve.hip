// gfx950 kernels of the equilibrium solve K u = f (arXiv 2505.02438,
// Sec. 2.2): a block-structured sparse product over the assembled CSR
// values and conjugate gradients preconditioned by the nodes' diagonal blocks (the iterative solver
// of the solver module, Sec. 3.2).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "block_sum.h"
#include "internal.h"
#include "kernels.h"

namespace soptx {

namespace {

// ------------------------------------------------------- solve (CG)
//
// The equilibrium system K u = f of the compliance problem, solved by
// conjugate gradients with a node-block Jacobi preconditioner on the assembled CSR values.
// In the iteration every product that is added to a sum is an fma, written out:
// the kernels of both its forms round alike, whatever the compiler would contract.
//
// y = K x.  K is a sum of DIM x DIM blocks, so a node's DIM rows share one
// neighbour list: row DIM I + a holds, for neighbour J = nb(I)[q], the
// entries of columns DIM J .. DIM J + DIM - 1 at row_ptr[DIM I + a] + DIM q.
// The kernel reads the neighbour lists (one id per block) instead of the
// column indices.  L lanes per node; lane s takes q = s, s + L, ...; the L
// partial sums of a row are added by an xor tree (a fixed order).  With
// xy_part, also the block partial of sum_r x_r y_r.
template <int DIM, int L>
__global__ __launch_bounds__(256) void k_spmv(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ nb,
                                              const double *__restrict__ K, const double *__restrict__ x,
                                              double *__restrict__ y, double *__restrict__ xy_part,
                                              int64_t n_nodes) {
    __shared__ double red[256];
    const int sub = threadIdx.x % L;
    const int64_t I = ((int64_t)blockIdx.x * 256 + threadIdx.x) / L;
    double acc[DIM];
#pragma unroll
    for (int a = 0; a < DIM; a++) acc[a] = 0.0;
    if (I < n_nodes) {
        const int b = row_ptr[DIM * I];
        const int rl = row_ptr[DIM * I + 1] - b;
        const int deg = rl / DIM;
        const int nbo = b / (DIM * DIM);
        for (int q = sub; q < deg; q += L) {
            const int J = nb[nbo + q];
            double xj[DIM];
#pragma unroll
            for (int e = 0; e < DIM; e++) xj[e] = x[(int64_t)DIM * J + e];
#pragma unroll
            for (int a = 0; a < DIM; a++)
#pragma unroll
                for (int e = 0; e < DIM; e++) acc[a] = fma(K[b + a * rl + DIM * q + e], xj[e], acc[a]);
        }
    }
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1)
#pragma unroll
        for (int a = 0; a < DIM; a++) acc[a] += __shfl_xor(acc[a], off);
    double xy = 0.0;
    if (I < n_nodes && sub == 0) {
#pragma unroll
        for (int a = 0; a < DIM; a++) {
            y[DIM * I + a] = acc[a];
            xy = fma(x[DIM * I + a], acc[a], xy);
        }
    }
    if (!xy_part) return;
    const double bs = block_sum_256(xy, red);
    if (threadIdx.x == 0) xy_part[blockIdx.x] = bs;
}

// Node-block Jacobi preconditioner: binv[I] = the inverse of node I's
// DIM x DIM diagonal block of K (row-major), by the adjugate.  A singular
// block (an isolated node) gives the inverse of its diagonal, 0 where that
// is 0, so such dofs stay put.
template <int DIM>
__global__ __launch_bounds__(256) void k_block_inv(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ nb,
                                                   const double *__restrict__ K, double *__restrict__ binv,
                                                   int64_t n_nodes) {
    const int64_t I = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (I >= n_nodes) return;
    const int b0 = row_ptr[DIM * I];
    const int rl = row_ptr[DIM * I + 1] - b0;
    const int nbo = b0 / (DIM * DIM);
    double B[DIM][DIM];
#pragma unroll
    for (int a = 0; a < DIM; a++)
#pragma unroll
        for (int c = 0; c < DIM; c++) B[a][c] = 0.0;
    for (int q = 0; q < rl / DIM; q++)
        if (nb[nbo + q] == I) {
#pragma unroll
            for (int a = 0; a < DIM; a++)
#pragma unroll
                for (int c = 0; c < DIM; c++) B[a][c] = K[b0 + a * rl + DIM * q + c];
        }
    double X[DIM][DIM];
    double det;
    if (DIM == 2) {
        det = B[0][0] * B[1][1] - B[0][1] * B[1][0];
        X[0][0] = B[1][1];
        X[0][1] = -B[0][1];
        X[1][0] = -B[1][0];
        X[1][1] = B[0][0];
    } else {
        X[0][0] = B[1][1] * B[2][2] - B[1][2] * B[2][1];
        X[0][1] = B[0][2] * B[2][1] - B[0][1] * B[2][2];
        X[0][2] = B[0][1] * B[1][2] - B[0][2] * B[1][1];
        X[1][0] = B[1][2] * B[2][0] - B[1][0] * B[2][2];
        X[1][1] = B[0][0] * B[2][2] - B[0][2] * B[2][0];
        X[1][2] = B[0][2] * B[1][0] - B[0][0] * B[1][2];
        X[2][0] = B[1][0] * B[2][1] - B[1][1] * B[2][0];
        X[2][1] = B[0][1] * B[2][0] - B[0][0] * B[2][1];
        X[2][2] = B[0][0] * B[1][1] - B[0][1] * B[1][0];
        det = B[0][0] * X[0][0] + B[0][1] * X[1][0] + B[0][2] * X[2][0];
    }
    double *o = binv + (int64_t)DIM * DIM * I;
    if (det != 0.0 && det == det) {
        const double id = 1.0 / det;
#pragma unroll
        for (int a = 0; a < DIM; a++)
#pragma unroll
            for (int c = 0; c < DIM; c++) o[a * DIM + c] = X[a][c] * id;
    } else {
#pragma unroll
        for (int a = 0; a < DIM; a++)
#pragma unroll
            for (int c = 0; c < DIM; c++) o[a * DIM + c] = (a == c && B[a][a] != 0.0) ? 1.0 / B[a][a] : 0.0;
    }
}

// One node's CG vector step (mode 0: r = f - q, p = z; mode 1: u += al p,
// r -= al q), then z = B^-1 r and the node's terms of r.z and r.r in dof order.
template <int DIM>
__device__ __forceinline__ void cg_node(int mode, double al, int64_t I, const double *__restrict__ f,
                                        double *__restrict__ u, double *__restrict__ r, double *__restrict__ z,
                                        double *__restrict__ p, const double *__restrict__ q,
                                        const double *__restrict__ binv, double &rz, double &rr) {
    const int64_t d0 = DIM * I;
    double ri[DIM];
    if (mode == 0) {
#pragma unroll
        for (int a = 0; a < DIM; a++) ri[a] = f[d0 + a] - q[d0 + a];
    } else {
#pragma unroll
        for (int a = 0; a < DIM; a++) {
            u[d0 + a] = fma(al, p[d0 + a], u[d0 + a]);
            ri[a] = fma(-al, q[d0 + a], r[d0 + a]);
        }
    }
    const double *bi = binv + (int64_t)DIM * DIM * I;
#pragma unroll
    for (int a = 0; a < DIM; a++) {
        double t = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; c++) t = fma(bi[a * DIM + c], ri[c], t);
        r[d0 + a] = ri[a];
        z[d0 + a] = t;
        if (mode == 0) p[d0 + a] = t;
        rz = fma(ri[a], t, rz);
        rr = fma(ri[a], ri[a], rr);
    }
}

// CG vector steps, one thread per node (its DIM dofs, so that z = B^-1 r
// uses the node's updated residual), block partials in a fixed order.
// Scalars sc: [0] r.z, [1] alpha, [2] beta, [3] r.r, [4] r0.r0, [5] p.q.
// mode 0 (start, q = K u): r = f - q, z = B^-1 r, p = z.
// mode 1 (iteration, q = K p): u += alpha p, r -= alpha q, z = B^-1 r.
// Both leave block partials of r.z (part[b]) and r.r (part[nb + b]); mode 0
// also of f.f (part[2 nb + b]).
template <int DIM>
__global__ __launch_bounds__(256) void k_cg_vec(int mode, const double *__restrict__ f, double *__restrict__ u,
                                                double *__restrict__ r, double *__restrict__ z,
                                                double *__restrict__ p, const double *__restrict__ q,
                                                const double *__restrict__ binv, const double *__restrict__ sc,
                                                double *__restrict__ part, int64_t n_nodes) {
    __shared__ double red[256];
    const int64_t I = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double rz = 0.0, rr = 0.0, ff = 0.0;
    if (I < n_nodes) {
        cg_node<DIM>(mode, mode == 0 ? 0.0 : sc[1], I, f, u, r, z, p, q, binv, rz, rr);
        if (mode == 0)
#pragma unroll
            for (int a = 0; a < DIM; a++) ff += f[DIM * I + a] * f[DIM * I + a];
    }
    const double brz = block_sum_256(rz, red);
    const double brr = block_sum_256(rr, red);
    const double bff = mode == 0 ? block_sum_256(ff, red) : 0.0;
    if (threadIdx.x == 0) {
        part[blockIdx.x] = brz;
        part[gridDim.x + blockIdx.x] = brr;
        if (mode == 0) part[2 * gridDim.x + blockIdx.x] = bff;
    }
}

// p = z + beta p
__global__ __launch_bounds__(256) void k_cg_p(double *__restrict__ p, const double *__restrict__ z,
                                              const double *__restrict__ sc, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = fma(sc[2], p[i], z[i]);
}

// ---- The iteration of small systems: two launches.
//
// k_cg_step_spmv forms beta and p = z + beta p (at every gathered node, the
// node's own into the other of two p buffers) and q = K p with the partials of
// p.q; k_cg_step_vec forms alpha, then u, r, z and the partials of r.z and r.r.
// Every block adds the partials of the launch before it, in the order of
// k_cg_scalars, so that no launch is needed for the two scalars; the sums and
// every product are those of the separate kernels above, bit for bit.  At
// these sizes an iteration is launches and chains of loads: K is read from
// the last-level cache.  So what the scalar does not touch (K, the neighbours'
// z and p, the node's own vectors) is read ahead of the partials.
// 120x40x8 hexahedra (133,947 dofs), per iteration: 18.5 + 5.5 us, 24.2 in all,
// against three launches of 16.2, 8.1 and 4.7 us and a host read every 8
// iterations (32.3); the 150x50 quadrilaterals 4.3 + 3.0 us, 8.2 in all, against
// 3.7, 4.8 and 3.6 us (18.3; there the host's 3.7 us per launch are the floor).
// In the first launch K is 75 MB of loads, each line touched by two of them:
// with non-temporal loads (no reuse in the first cache) it takes 28 us; K
// through LDS in whole lines 25, z and p side by side 19.6, one neighbour ahead
// instead of two 20.7, a contiguous eighth of the nodes per XCD 19.2, every wave
// adding the partials itself (no barrier) 22.
//
// The residual is checked on the device every kCgCheck iterations, by block 0
// of the launch that starts the next one; launches after a stop return at
// once, so the host can enqueue ahead instead of waiting for each check.  fin:
// [0] stopped, [1] iterations, [2] r.r.

// x + its DPP partner
template <int CTRL>
__device__ __forceinline__ double add_dpp(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return x + __hiloint2double(hi, lo);
}

// N sums over a block of 256 threads, each in block_sum_256's order, returned
// to every thread, with one barrier (two where red is reused: `again`): every
// wave adds the 256 values itself, lane l the sixteen l + 16 j (the tree's
// first four levels), then the rest within a row of 16 lanes.
template <int N>
__device__ __forceinline__ void block_sums_256(double (&x)[N], double (*red)[256], bool again) {
    if (again) __syncthreads();
#pragma unroll
    for (int k = 0; k < N; k++) red[k][threadIdx.x] = x[k];
    __syncthreads();
    const int l = threadIdx.x & 15;
#pragma unroll
    for (int k = 0; k < N; k++) {
        double v[16];
#pragma unroll
        for (int j = 0; j < 16; j++) v[j] = red[k][l + 16 * j];
#pragma unroll
        for (int st = 8; st > 0; st >>= 1)
#pragma unroll
            for (int j = 0; j < st; j++) v[j] += v[j + st];
        double t = add_dpp<0x108>(v[0]);  // row_shl: lane l + 8, 4, 2, 1
        t = add_dpp<0x104>(t);
        t = add_dpp<0x102>(t);
        t = add_dpp<0x101>(t);
        x[k] = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(t)),
                                __builtin_amdgcn_readfirstlane(__double2loint(t)));
    }
}

// Thread t's share of the sum of n block partials in the order of k_cg_scalars
// (1024 strided sums, then a halving tree): the strided sums t, t + 256, t +
// 512 and t + 768 and the tree's first two levels; block_sums_256 does the
// rest.
template <int ROUNDS>
__device__ __forceinline__ double scalar_share(const double *__restrict__ part, int n) {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    // ROUNDS rounds of loads in flight together, then added in order
    for (int k0 = threadIdx.x; k0 < n; k0 += ROUNDS * 1024) {
        double x[ROUNDS][4];
#pragma unroll
        for (int h = 0; h < ROUNDS; h++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int k = k0 + 256 * g + 1024 * h;
                x[h][g] = k < n ? part[k] : 0.0;
            }
#pragma unroll
        for (int h = 0; h < ROUNDS; h++)
#pragma unroll
            for (int g = 0; g < 4; g++)
                if (k0 + 256 * g + 1024 * h < n) v[g] += x[h][g];
    }
    v[0] += v[2];
    v[1] += v[3];
    return v[0] + v[1];
}

// sum over the L lanes of a node by the xor tree of k_spmv
template <int L>
__device__ __forceinline__ double lanes_sum(double x) {
    static_assert(L == 16 || L == 8, "rows of 16 or 8 lanes");
    if (L == 16) {
        // a rotation by half the period is the xor partner
        x = add_dpp<0x128>(x);
        x = add_dpp<0x124>(x);
        x = add_dpp<0x122>(x);
        return add_dpp<0x121>(x);
    }
    // xor 4: mirror within 8 lanes (xor 7), then reverse each quad (xor 3)
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x141, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x141, 0xf, 0xf, true);
    lo = __builtin_amdgcn_update_dpp(0, lo, 0x1b, 0xf, 0xf, true);
    hi = __builtin_amdgcn_update_dpp(0, hi, 0x1b, 0xf, 0xf, true);
    x += __hiloint2double(hi, lo);
    x = add_dpp<0x4e>(x);     // quad lanes 2 3 0 1: xor 2
    return add_dpp<0xb1>(x);  // quad lanes 1 0 3 2: xor 1
}

template <int DIM, int L>
__global__ __launch_bounds__(256) void k_cg_step_spmv(CgStep A, int it, bool check) {
    __shared__ double red[1][256];
    // Looked at before the first write: nothing waits for it alone.  In a launch
    // that checks only block 0, which may write the stop, looks at it (all its
    // waves before the barrier ahead of that write); the other blocks would find
    // it or not by when they run, and work on, into buffers that nothing reads
    // after a stop.
    const bool stopped = (!check || blockIdx.x == 0) && A.fin[0] != 0.0;
    const bool first = it == 0;  // p = z
    const double *__restrict__ z = A.z;
    const double *__restrict__ po = A.p[(it & 1) ^ 1];
    double *__restrict__ pn = A.p[it & 1];
    const int sub = threadIdx.x % L;
    const int64_t I = ((int64_t)blockIdx.x * 256 + threadIdx.x) / L;
    const bool live = I < A.n_nodes;
    const double old = first ? 1.0 : A.sc[8 * ((it & 1) ^ 1)];
    const double share = first ? 0.0 : scalar_share<1>(A.rz_part, A.n_rz);
    // the lane's first kAhead neighbours and the node's own z and p
    constexpr int kAhead = 2;
    int b = 0, rl = 0, deg = 0, nbo = 0, J[kAhead];
    double Kv[kAhead][DIM][DIM], zj[kAhead][DIM], pj[kAhead][DIM], zi[DIM], pi[DIM];
    if (live) {
        b = A.row_ptr[DIM * I];
        rl = A.row_ptr[DIM * I + 1] - b;
        deg = rl / DIM;
        nbo = b / (DIM * DIM);
    }
#pragma unroll
    for (int h = 0; h < kAhead; h++) J[h] = sub + h * L < deg ? A.nb[nbo + sub + h * L] : -1;
#pragma unroll
    for (int h = 0; h < kAhead; h++)
        if (J[h] >= 0) {
#pragma unroll
            for (int a = 0; a < DIM; a++)
#pragma unroll
                for (int e = 0; e < DIM; e++) Kv[h][a][e] = A.K[b + a * rl + DIM * (sub + h * L) + e];
#pragma unroll
            for (int e = 0; e < DIM; e++) {
                zj[h][e] = z[(int64_t)DIM * J[h] + e];
                pj[h][e] = first ? 0.0 : po[(int64_t)DIM * J[h] + e];
            }
        }
    if (live && sub == 0)
#pragma unroll
        for (int a = 0; a < DIM; a++) {
            zi[a] = z[DIM * I + a];
            pi[a] = first ? 0.0 : po[DIM * I + a];
        }
    double beta = 0.0;
    if (!first) {
        double t[1] = {share};
        block_sums_256(t, red, false);
        beta = t[0] / old;
        if (blockIdx.x == 0 && !stopped) {
            if (threadIdx.x == 0) A.sc[8 * (it & 1)] = t[0];
            if (check) {
                double s[1] = {scalar_share<1>(A.rz_part + A.n_rz, A.n_rz)};
                block_sums_256(s, red, true);
                // stop: converged, or broke down (NaN)
                if (threadIdx.x == 0 && !(sqrt(s[0] / A.ref) > A.rtol)) {
                    A.fin[1] = A.host[1] = (double)it;
                    A.fin[2] = A.host[2] = s[0];
                    A.fin[0] = A.host[0] = 1.0;
                }
            }
        }
    }
    double acc[DIM];
#pragma unroll
    for (int a = 0; a < DIM; a++) acc[a] = 0.0;
#pragma unroll
    for (int h = 0; h < kAhead; h++)
        if (J[h] >= 0) {
            double x[DIM];
#pragma unroll
            for (int e = 0; e < DIM; e++) x[e] = first ? zj[h][e] : fma(beta, pj[h][e], zj[h][e]);
#pragma unroll
            for (int a = 0; a < DIM; a++)
#pragma unroll
                for (int e = 0; e < DIM; e++) acc[a] = fma(Kv[h][a][e], x[e], acc[a]);
        }
    for (int q = sub + kAhead * L; q < deg; q += L) {
        const int64_t d0 = (int64_t)DIM * A.nb[nbo + q];
        double x[DIM];
#pragma unroll
        for (int e = 0; e < DIM; e++) x[e] = first ? z[d0 + e] : fma(beta, po[d0 + e], z[d0 + e]);
#pragma unroll
        for (int a = 0; a < DIM; a++)
#pragma unroll
            for (int e = 0; e < DIM; e++) acc[a] = fma(A.K[b + a * rl + DIM * q + e], x[e], acc[a]);
    }
#pragma unroll
    for (int a = 0; a < DIM; a++) acc[a] = lanes_sum<L>(acc[a]);
    if (stopped) return;
    double xy[1] = {0.0};
    if (live && sub == 0) {
#pragma unroll
        for (int a = 0; a < DIM; a++) {
            const double x = first ? zi[a] : fma(beta, pi[a], zi[a]);
            pn[DIM * I + a] = x;
            A.q[DIM * I + a] = acc[a];
            xy[0] = fma(x, acc[a], xy[0]);
        }
    }
    block_sums_256(xy, red, !first);
    if (threadIdx.x == 0) A.pq_part[blockIdx.x] = xy[0];
}

template <int DIM>
__global__ __launch_bounds__(256) void k_cg_step_vec(CgStep A, int it) {
    __shared__ double red[2][256];
    const bool stopped = A.fin[0] != 0.0;
    const int64_t I = (int64_t)blockIdx.x * 256 + threadIdx.x, d0 = DIM * I;
    const bool live = I < A.n_nodes;
    const double *__restrict__ p = A.p[it & 1];
    double uu[DIM], rr[DIM], pp[DIM], qq[DIM], bi[DIM * DIM];
    if (live) {
#pragma unroll
        for (int a = 0; a < DIM; a++) {
            uu[a] = A.u[d0 + a];
            rr[a] = A.r[d0 + a];
            pp[a] = p[d0 + a];
            qq[a] = A.q[d0 + a];
        }
#pragma unroll
        for (int c = 0; c < DIM * DIM; c++) bi[c] = A.binv[DIM * DIM * I + c];
    }
    const double rz = A.sc[8 * (it & 1)];
    double t[1] = {scalar_share<4>(A.pq_part, A.n_pq)};
    block_sums_256(t, red, false);
    if (stopped) return;
    const double al = rz / t[0];
    double s[2] = {0.0, 0.0};  // r.z, r.r
    if (live) {
        double ri[DIM];
#pragma unroll
        for (int a = 0; a < DIM; a++) {
            A.u[d0 + a] = fma(al, pp[a], uu[a]);
            ri[a] = fma(-al, qq[a], rr[a]);
        }
#pragma unroll
        for (int a = 0; a < DIM; a++) {
            double v = 0.0;
#pragma unroll
            for (int c = 0; c < DIM; c++) v = fma(bi[a * DIM + c], ri[c], v);
            A.r[d0 + a] = ri[a];
            A.z[d0 + a] = v;
            s[0] = fma(ri[a], v, s[0]);
            s[1] = fma(ri[a], ri[a], s[1]);
        }
    }
    block_sums_256(s, red, true);
    if (threadIdx.x == 0) {
        A.rz_part[blockIdx.x] = s[0];
        A.rz_part[A.n_rz + blockIdx.x] = s[1];
    }
}

__global__ void k_cg_clear(double *x, int n) {
    if ((int)threadIdx.x < n) x[threadIdx.x] = 0.0;
}

// r.r after the last iteration, where no check stopped earlier
__global__ __launch_bounds__(256) void k_cg_step_end(CgStep A, int it) {
    __shared__ double red[1][256];
    if (A.fin[0] != 0.0) return;
    double s[1] = {scalar_share<1>(A.rz_part + A.n_rz, A.n_rz)};
    block_sums_256(s, red, false);
    if (threadIdx.x == 0) {
        A.host[1] = (double)it;
        A.host[2] = s[0];
        A.host[0] = 1.0;
    }
}

// One block of kScalThreads: sums of n block partials, thread t taking
// k = t, t + kScalThreads, ... in order, then a fixed tree.
// what 0 (start):     r.z and r.r from part -> sc[0], sc[3], sc[4] = sc[3]
// what 3 (start):     f.f from part -> sc[6]
// what 1 (alpha):     p.q from part -> sc[5], sc[1] = sc[0] / p.q
// what 2 (beta):      r.z, r.r from part -> sc[2] = new r.z / sc[0], sc[0], sc[3]
constexpr int kScalThreads = 1024;
__global__ __launch_bounds__(kScalThreads) void k_cg_scalars(int what, const double *__restrict__ part, int n,
                                                             double *sc) {
    __shared__ double red[2][kScalThreads];
    double t0 = 0.0, t1 = 0.0;
    for (int k = threadIdx.x; k < n; k += kScalThreads) {
        t0 += part[k];
        if (what != 1 && what != 3) t1 += part[n + k];
    }
    red[0][threadIdx.x] = t0;
    red[1][threadIdx.x] = t1;
    __syncthreads();
    for (int st = kScalThreads / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            red[0][threadIdx.x] += red[0][threadIdx.x + st];
            red[1][threadIdx.x] += red[1][threadIdx.x + st];
        }
        __syncthreads();
    }
    t0 = red[0][0];
    t1 = red[1][0];
    if (threadIdx.x != 0) return;
    if (what == 3) {
        sc[6] = t0;
    } else if (what == 0) {
        sc[0] = t0;
        sc[3] = t1;
        sc[4] = t1;
    } else if (what == 1) {
        sc[5] = t0;
        sc[1] = sc[0] / t0;
    } else {
        sc[2] = t0 / sc[0];
        sc[0] = t0;
        sc[3] = t1;
    }
}

}  // namespace

// ---------------------------------------------------------------- launchers

int64_t spmv_blocks(int dim, int64_t n_nodes) {
    const int L = dim == 3 ? 16 : 8;
    return (n_nodes * L + 255) / 256;
}

hipError_t launch_spmv(int dim, const int32_t *row_ptr, const int32_t *nb, const double *K, const double *x,
                       double *y, double *xy_part, int64_t n_nodes, hipStream_t st) {
    const unsigned g = (unsigned)spmv_blocks(dim, n_nodes);
    if (g == 0) return hipSuccess;
    if (dim == 3) hipLaunchKernelGGL((k_spmv<3, 16>), dim3(g), dim3(256), 0, st, row_ptr, nb, K, x, y, xy_part, n_nodes);
    else hipLaunchKernelGGL((k_spmv<2, 8>), dim3(g), dim3(256), 0, st, row_ptr, nb, K, x, y, xy_part, n_nodes);
    return hipGetLastError();
}

int64_t cg_vec_blocks(int dim, int64_t ndof) { return (ndof / dim + 255) / 256; }

hipError_t launch_block_inv(int dim, const int32_t *row_ptr, const int32_t *nb, const double *K, double *binv,
                            int64_t n_nodes, hipStream_t st) {
    const unsigned g = (unsigned)((n_nodes + 255) / 256);
    if (g == 0) return hipSuccess;
    if (dim == 3) hipLaunchKernelGGL(k_block_inv<3>, dim3(g), dim3(256), 0, st, row_ptr, nb, K, binv, n_nodes);
    else hipLaunchKernelGGL(k_block_inv<2>, dim3(g), dim3(256), 0, st, row_ptr, nb, K, binv, n_nodes);
    return hipGetLastError();
}

hipError_t launch_cg_vec(int dim, int mode, const double *f, double *u, double *r, double *z, double *p,
                         const double *q, const double *binv, const double *sc, double *part, int64_t ndof,
                         hipStream_t st) {
    const unsigned g = (unsigned)cg_vec_blocks(dim, ndof);
    if (g == 0) return hipSuccess;
    if (dim == 3)
        hipLaunchKernelGGL(k_cg_vec<3>, dim3(g), dim3(256), 0, st, mode, f, u, r, z, p, q, binv, sc, part, ndof / 3);
    else
        hipLaunchKernelGGL(k_cg_vec<2>, dim3(g), dim3(256), 0, st, mode, f, u, r, z, p, q, binv, sc, part, ndof / 2);
    return hipGetLastError();
}

hipError_t launch_cg_step(int dim, const CgStep &A, int it, bool check, hipStream_t st) {
    const unsigned g = (unsigned)spmv_blocks(dim, A.n_nodes);
    if (g == 0) return hipErrorInvalidValue;
    if (dim == 3) hipLaunchKernelGGL((k_cg_step_spmv<3, 16>), dim3(g), dim3(256), 0, st, A, it, check);
    else hipLaunchKernelGGL((k_cg_step_spmv<2, 8>), dim3(g), dim3(256), 0, st, A, it, check);
    return hipGetLastError();
}

hipError_t launch_cg_step_vec(int dim, const CgStep &A, int it, hipStream_t st) {
    const unsigned g = (unsigned)A.n_rz;
    if (dim == 3) hipLaunchKernelGGL(k_cg_step_vec<3>, dim3(g), dim3(256), 0, st, A, it);
    else hipLaunchKernelGGL(k_cg_step_vec<2>, dim3(g), dim3(256), 0, st, A, it);
    return hipGetLastError();
}

hipError_t launch_cg_clear(double *x, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_cg_clear, dim3(1), dim3(64), 0, st, x, n);
    return hipGetLastError();
}

hipError_t launch_cg_step_end(const CgStep &A, int it, hipStream_t st) {
    hipLaunchKernelGGL(k_cg_step_end, dim3(1), dim3(256), 0, st, A, it);
    return hipGetLastError();
}

hipError_t launch_cg_p(double *p, const double *z, const double *sc, int64_t n, hipStream_t st) {
    const unsigned g = (unsigned)((n + 255) / 256);
    if (g == 0) return hipSuccess;
    hipLaunchKernelGGL(k_cg_p, dim3(g), dim3(256), 0, st, p, z, sc, n);
    return hipGetLastError();
}

hipError_t launch_cg_scalars(int what, const double *part, int n, double *sc, hipStream_t st) {
    hipLaunchKernelGGL(k_cg_scalars, dim3(1), dim3(kScalThreads), 0, st, what, part, n, sc);
    return hipGetLastError();
}

}  // namespace soptx
