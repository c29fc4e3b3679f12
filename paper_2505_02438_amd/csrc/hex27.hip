// gfx950 kernels of the fused assembly of Q2 hexahedra (27 nodes, 3 x 3 x 3
// Gauss points, straight or curved; arXiv 2505.02438, Sec. 2.2): K by row
// groups (HostPlan::rg_*), no element matrix in memory.
//
// The element-matrix form (k_ke_general_wide, k_gather_general) writes 1.26 GB
// of element matrices, reads them back through a 170 MB table and then writes
// K: 464 + 526 us on the curved 60 x 20 x 20 mesh (24,000 elements, 898 MB of
// K), where K alone takes about 140 us.  Here a workgroup owns the rows of a
// few nodes (8 on a mesh of boxes) and walks the Gauss points of the (8)
// elements around them together, so every block of K is formed on chip and
// written once, in whole rows.  The price is arithmetic: the rows of an
// element are formed by the owners of its nodes, so block (i, j) and its
// transpose are both computed (4.3e9 FMAs of gradient products there), and the
// gradients at the points are formed 8 times over (1.3e9).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "internal.h"
#include "kernels.h"

namespace soptx {

namespace {

constexpr int kThreads = 128;
constexpr int kNQ = 27;            // Gauss points: qx + 3 qy + 9 qz
// nine values padded to ten, so that they move in 16-byte pieces: the geometry
// of a point, and the gradients of a line of three nodes
constexpr int kTen = 10;
constexpr int kGeo = kTen * kNQ;   // doubles of geometry per element
// gradients of one step: [visit][qx][line][10]
constexpr int kVisit = 3 * 9 * kTen;
constexpr int kStep = kRgVisits * kVisit;
static_assert(2 * kStep <= kRgStage, "two steps' gradients lie in the stage");
static_assert(kRgPairs * 9 <= kThreads, "a lane per pair and three columns");
static_assert(4 * kRgRows <= kThreads, "a thread per row value");

typedef double d2 __attribute__((ext_vector_type(2)));

// 1D quadratic Lagrange basis on {0, 1/2, 1} and its derivative
__host__ __device__ constexpr double lag(int k, double t) {
    return k == 0 ? (1.0 - t) * (1.0 - 2.0 * t) : k == 1 ? 4.0 * t * (1.0 - t) : t * (2.0 * t - 1.0);
}
__host__ __device__ constexpr double dlag(int k, double t) {
    return k == 0 ? 4.0 * t - 3.0 : k == 1 ? 4.0 - 8.0 * t : 4.0 * t - 1.0;
}
constexpr double kRoot35 = 0.77459666924148337703585307995648;  // sqrt(3/5)
__host__ __device__ constexpr double point(int q) { return 0.5 * (1.0 + (q - 1) * kRoot35); }
__host__ __device__ constexpr double weight(int q) { return q == 1 ? 4.0 / 9.0 : 5.0 / 18.0; }

// per-mesh geometry, once per pattern: geo[e][q][3 m + a] = sqrt(w_q |det J_q|)
// d xi_m / d x_a (padded to ten), one thread per (element, point)
__global__ __launch_bounds__(256) void k_hex27_geometry(const int32_t *__restrict__ cells,
                                                        const double *__restrict__ coords, int64_t n_cells,
                                                        double *__restrict__ geo) {
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n_cells * kNQ) return;
    const int64_t e = x / kNQ;
    const int q = (int)(x - e * kNQ);
    const double t[3] = {point(q % 3), point(q / 3 % 3), point(q / 9)};
    double J[3][3] = {};  // d x_a / d xi_m
    for (int i = 0; i < 27; i++) {
        // lattice position of local node i: the 8 corners, then the others in
        // ascending a + 3 b + 9 c
        int l[3];
        if (i < 8) {
            l[0] = 2 * ((i ^ (i >> 1)) & 1);
            l[1] = i & 2;
            l[2] = (i & 4) / 2;
        } else {
            // the (i - 8)-th lattice point with an odd coordinate
            int s = 0, n = i - 8;
            for (; s < 27; s++) {
                const bool odd = s % 3 == 1 || s / 3 % 3 == 1 || s / 9 == 1;
                if (odd && n-- == 0) break;
            }
            l[0] = s % 3;
            l[1] = s / 3 % 3;
            l[2] = s / 9;
        }
        double f[3], d[3];
#pragma unroll
        for (int m = 0; m < 3; m++) {
            f[m] = lag(l[m], t[m]);
            d[m] = dlag(l[m], t[m]);
        }
        const double g[3] = {d[0] * f[1] * f[2], f[0] * d[1] * f[2], f[0] * f[1] * d[2]};
        const int64_t n = cells[e * 27 + i];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const double xa = coords[3 * n + a];
#pragma unroll
            for (int m = 0; m < 3; m++) J[a][m] = fma(xa, g[m], J[a][m]);
        }
    }
    const double c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1], c01 = J[0][2] * J[2][1] - J[0][1] * J[2][2],
                 c02 = J[0][1] * J[1][2] - J[0][2] * J[1][1], c10 = J[1][2] * J[2][0] - J[1][0] * J[2][2],
                 c11 = J[0][0] * J[2][2] - J[0][2] * J[2][0], c12 = J[0][2] * J[1][0] - J[0][0] * J[1][2],
                 c20 = J[1][0] * J[2][1] - J[1][1] * J[2][0], c21 = J[0][1] * J[2][0] - J[0][0] * J[2][1],
                 c22 = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    const double det = J[0][0] * c00 + J[0][1] * c10 + J[0][2] * c20;
    const double s = sqrt(weight(q % 3) * weight(q / 3 % 3) * weight(q / 9) * fabs(det)) / det;
    double *o = geo + x * kTen;
    o[0] = s * c00; o[1] = s * c01; o[2] = s * c02;
    o[3] = s * c10; o[4] = s * c11; o[5] = s * c12;
    o[6] = s * c20; o[7] = s * c21; o[8] = s * c22;
    o[9] = 0.0;
}

__device__ __noinline__ double hex27_pow(double x, double p) { return pow(x, p); }

// wave-uniform reads of the plan's tables, through the scalar cache
__device__ __forceinline__ int table(const int32_t *p, int64_t i) {
    return ((const __attribute__((address_space(4))) int32_t *)p)[i];
}

// One workgroup of two waves per row group, four per CU (40 KB of LDS).
//
// Nine steps of three points (one line of the rule along x): the gradients of
// the next step's points, sqrt(w |det J|) J^-T grad phi_k for all 27 nodes of
// every visited element, go to LDS while the products of this one are formed
// (two buffers, one barrier a step).  A thread of the gradients has one
// (visit, qx) and a line of three nodes along x: 30 FP64 operations for 9
// values by the tensor product, from geometry read a step ahead.  A lane of
// the products has a pair of rows (two of the group's nodes in one element)
// and three columns: 15 LDS values for 54 FMAs a point, the six 3 x 3 sums in
// registers through all 27 points, so that nothing is added in LDS meanwhile.
// At the end E and L are applied (both are linear) and the blocks go to the
// rows in LDS, over the gradients, in the order of the visits (ascending
// element): first terms, second terms, then any more from slots; and the rows
// leave as whole runs by non-temporal stores.
//
// Measured on the curved 60 x 20 x 20 mesh, back to back: 543 us on the same
// inputs (tables and geometry, 109 MB, in the last-level cache), 602 with three
// patterns in turn, against the 990 of the element-matrix form (renumbered at
// random 569 against 996; 2,000 elements 66 against 95, 36 elements 16 against
// 18); under the profiler 594 to 664.  Vector instructions take half the issue
// cycles (58 of 100 are FMAs), LDS 57 %: with two waves per SIMD (256 VGPRs)
// neither is reached.  On the way: three workgroups per CU with a slot for every further
// term 690 us; the terms added rank by rank 585; 8-byte instead of 16-byte LDS
// moves of the gradients 15 us more; four waves a workgroup sharing the points,
// and persistent workgroups that read the next group's tables ahead, spill
// (1,090 and 1,150).
__global__ __launch_bounds__(kThreads, 2) void k_assemble_hex27(Hex27Params P) {
    __shared__ __align__(16) double lds[kRgStage];
    __shared__ double tl[3][3], td[3][3];  // basis and derivative [node][point]
    __shared__ double sE[kRgVisits];
    __shared__ int32_t srow[kRgRows][4];
    const int tid = threadIdx.x;
    // windows of groups dealt to the XCDs in contiguous runs, so that groups
    // that visit the same elements meet in one L2
    const int bid = blockIdx.x, W = P.window, base = bid - bid % W;
    const int64_t g = base + W <= P.n_groups ? base + (bid % 8) * (W / 8) + (bid - base) / 8 : bid;
    // the group's tables, indexed by it alone so that they are read together;
    // the lane's pair and columns
    const int pt = tid / 9, jt = tid - 9 * pt, ptc = pt < kRgPairs ? pt : 0;
    const int nr = table(P.info, 4 * g), np = table(P.info, 4 * g + 1), stage = table(P.info, 4 * g + 2),
              nx = table(P.info, 4 * g + 3);
    const int c0 = P.pairs[2 * (g * kRgPairs + ptc)], c1 = P.pairs[2 * (g * kRgPairs + ptc) + 1];
    int codes[3];  // of the two rows' blocks, 16 bits each
#pragma unroll
    for (int j = 0; j < 3; j++)
        codes[j] = P.code[(g * kRgPairs + ptc) * 54 + 3 * jt + j] |
                   (int)P.code[(g * kRgPairs + ptc) * 54 + 27 + 3 * jt + j] << 16;
    // a thread per entry of a block of three or more terms
    constexpr int kExtLoads = (9 * kRgExt + kThreads - 1) / kThreads;
    int exat[kExtLoads], exm[kExtLoads];  // read at the start, used at the end
#pragma unroll
    for (int x = 0; x < kExtLoads; x++) {
        const int k = (tid + x * kThreads) / 9;
        exat[x] = k < kRgExt ? P.ext[2 * (g * kRgExt + k)] : 0;
        exm[x] = k < kRgExt ? P.ext[2 * (g * kRgExt + k) + 1] : 0;
    }
    if (tid < 4 * kRgRows) (&srow[0][0])[tid] = P.rows[g * (4 * kRgRows) + tid];
    if (tid < kRgVisits) {
        const double r = P.rho[P.vis[g * kRgVisits + tid]];
        double t = 1.0;
        if (P.ip >= 0)
            for (int k = 0; k < P.ip; k++) t *= r;
        else t = hex27_pow(r, P.p);
        sE[tid] = P.Emin + t * (P.E0 - P.Emin);
    }
    if (tid < 9) {
        // constant indices: the tables are compile-time values
        double v = 0.0, d = 0.0;
#pragma unroll
        for (int x = 0; x < 9; x++)
            if (x == tid) {
                v = lag(x / 3, point(x % 3));
                d = dlag(x / 3, point(x % 3));
            }
        tl[tid / 3][tid % 3] = v;
        td[tid / 3][tid % 3] = d;
    }
    // the gradients' lane: nodes (kx = 0 .. 2, ky, kz) at point qx of visits gv and gv + 4
    const int yz = tid % 9, ky = yz % 3, kz = yz / 3, qx = tid / 9 % 3, gv = tid / 27;
    static_assert(kRgVisits == 8, "two visits per gradient thread");
    const d2 *geo[2];
    d2 J[2][5];
#pragma unroll
    for (int h = 0; h < 2; h++)
        geo[h] = reinterpret_cast<const d2 *>(P.geo + (int64_t)P.vis[g * kRgVisits + gv % 4 + 4 * h] * kGeo + qx * kTen);
    auto load_geo = [&](int s) {
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int x = 0; x < 5; x++) J[h][x] = geo[h][s * (3 * kTen / 2) + x];
    };
    load_geo(0);
    __syncthreads();
    double fx[3], dx[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        fx[k] = tl[k][qx];
        dx[k] = td[k][qx];
    }
    auto gradients = [&](int s, double *dst) {
        const int qy = s % 3, qz = s / 3;
        const double fy = tl[ky][qy], dy = td[ky][qy], fz = tl[kz][qz], dz = td[kz][qz];
        const double yzf = fy * fz, ydz = dy * fz, zdy = fy * dz;
        if (gv < 4) {
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int v = gv + 4 * h;
                const double j[9] = {J[h][0].x, J[h][0].y, J[h][1].x, J[h][1].y, J[h][2].x,
                                     J[h][2].y, J[h][3].x, J[h][3].y, J[h][4].x};
                double o[kTen];
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    const double A = yzf * j[a], B = fma(ydz, j[3 + a], zdy * j[6 + a]);
#pragma unroll
                    for (int k = 0; k < 3; k++) o[3 * k + a] = fma(dx[k], A, fx[k] * B);
                }
                o[9] = 0.0;
                d2 *w = reinterpret_cast<d2 *>(dst + v * kVisit + (qx * 9 + yz) * kTen);
#pragma unroll
                for (int x = 0; x < 5; x++) w[x] = d2{o[2 * x], o[2 * x + 1]};
            }
        }
    };
    struct Ops {
        double w[2][3], g[kTen];
    };
    const bool mine = pt < np;
    const int pv = mine ? c0 & 255 : 0, i0 = (c0 >> 8) & 255, i1x = c0 >> 16;
    const bool two = mine && i1x != 255;
    const int i1 = two ? i1x : i0;
    const int at0 = i0 / 3 * kTen + i0 % 3 * 3, at1 = i1 / 3 * kTen + i1 % 3 * 3;
    double acc[2][3][3][3];
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int a = 0; a < 3; a++)
#pragma unroll
                for (int c = 0; c < 3; c++) acc[r][j][a][c] = 0.0;
    auto load = [&](const double *gq, Ops &o) {
#pragma unroll
        for (int x = 0; x < 5; x++) {
            const d2 y = reinterpret_cast<const d2 *>(gq + kTen * jt)[x];
            o.g[2 * x] = y.x;
            o.g[2 * x + 1] = y.y;
        }
#pragma unroll
        for (int a = 0; a < 3; a++) {
            o.w[0][a] = gq[at0 + a];
            o.w[1][a] = gq[at1 + a];
        }
    };
    auto add = [&](const Ops &o) {
#pragma unroll
        for (int r = 0; r < 2; r++)
#pragma unroll
            for (int j = 0; j < 3; j++)
#pragma unroll
                for (int a = 0; a < 3; a++)
#pragma unroll
                    for (int c = 0; c < 3; c++) acc[r][j][a][c] = fma(o.w[r][a], o.g[3 * j + c], acc[r][j][a][c]);
    };
    gradients(0, lds);
    load_geo(1);
    __syncthreads();
    for (int s = 0; s < 9; s++) {
        const double *cur = lds + (s & 1) * kStep + pv * kVisit;
        Ops a, b;  // a point's operands are read while the one before is added
        load(cur, a);
        if (s < 8) {
            gradients(s + 1, lds + ((s + 1) & 1) * kStep);
            load_geo(s < 7 ? s + 2 : 8);
        }
        load(cur + 9 * kTen, b);
        add(a);
        load(cur + 18 * kTen, a);
        add(b);
        add(a);
        __syncthreads();
    }
    // E and L, then the blocks to the stage (the geometry and the gradients
    // are done with): every block's first term to its place and the third
    // and later ones to slots, then the second terms, then the slots
    const double lam = P.lam * sE[pv], mu = P.mu * sE[pv];
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            double(&p)[3][3] = acc[r][j];
            const double mtr = mu * (p[0][0] + p[1][1] + p[2][2]);
#pragma unroll
            for (int a = 0; a < 3; a++) {
                p[a][a] = lam * p[a][a] + mu * p[a][a] + mtr;
#pragma unroll
                for (int c = a + 1; c < 3; c++) {
                    const double u = p[a][c], l = p[c][a];
                    p[a][c] = lam * u + mu * l;
                    p[c][a] = lam * l + mu * u;
                }
            }
        }
    double *rowp[2];
    int rl[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        const int32_t *rw = srow[r == 0 ? (c1 & 0xffff) : c1 >> 16];
        rl[r] = 3 * rw[1];
        rowp[r] = lds + rw[2];
    }
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const int code = codes[j] >> (16 * r) & 0xffff;
            const bool slot = code & kRgSlot;
            if ((r == 0 ? mine : two) && !(code & kRgSecond)) {
                double *o = slot ? lds + stage + 9 * (code & (kRgSlot - 1)) : rowp[r] + 3 * code;
                const int ld = slot ? 3 : rl[r];
#pragma unroll
                for (int x = 0; x < 9; x++) o[x / 3 * ld + x % 3] = acc[r][j][x / 3][x % 3];
            }
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const int code = codes[j] >> (16 * r) & 0xffff;
            if ((r == 0 ? mine : two) && (code & (kRgSlot | kRgSecond)) == kRgSecond) {
                double *o = rowp[r] + 3 * (code & (kRgSecond - 1));
                double v[9];
#pragma unroll
                for (int x = 0; x < 9; x++) v[x] = o[x / 3 * rl[r] + x % 3];
#pragma unroll
                for (int x = 0; x < 9; x++) o[x / 3 * rl[r] + x % 3] = v[x] + acc[r][j][x / 3][x % 3];
            }
        }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < kExtLoads; x++) {
        const int k = tid + x * kThreads, n = exm[x] >> 24;
        if (k < 9 * nx) {
            double *o = lds + exat[x] + k % 9 / 3 * (exm[x] & 0xfff) + k % 3;
            const double *src = lds + stage + 9 * (exm[x] >> 12 & 0xfff) + k % 9;
            double v = *o;
            for (int t = 0; t < n; t++) v += src[9 * t];
            *o = v;
        }
    }
    __syncthreads();
    // each wave every other row
    for (int r = tid / 64; r < nr; r += kThreads / 64) {
        const int n = 9 * srow[r][1];
        const double *src = lds + srow[r][2];
        double *dst = P.K + srow[r][0];
        for (int x0 = tid % 64; x0 < n; x0 += 9 * 64) {
            double v[9];
#pragma unroll
            for (int k = 0; k < 9; k++) v[k] = x0 + k * 64 < n ? src[x0 + k * 64] : 0.0;
#pragma unroll
            for (int k = 0; k < 9; k++)
                if (x0 + k * 64 < n) __builtin_nontemporal_store(v[k], dst + x0 + k * 64);
        }
    }
}

}  // namespace

hipError_t launch_hex27_geometry(const int32_t *cells, const double *coords, int64_t n_cells, double *geo,
                                 hipStream_t st) {
    if (n_cells <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_hex27_geometry, dim3((unsigned)((n_cells * kNQ + 255) / 256)), dim3(256), 0, st, cells, coords,
                       n_cells, geo);
    return hipGetLastError();
}

hipError_t launch_assemble_hex27(const Hex27Params &P0, hipStream_t st) {
    if (P0.n_groups <= 0) return hipSuccess;
    Hex27Params P = P0;
    P.window = std::max(8, 4 * (P.n_cu > 0 ? P.n_cu : 256) / 8 * 8);
    hipLaunchKernelGGL(k_assemble_hex27, dim3((unsigned)P.n_groups), dim3(kThreads), 0, st, P);
    return hipGetLastError();
}

}  // namespace soptx
