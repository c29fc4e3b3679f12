// gfx950 kernels of the optimality-criteria update (arXiv 2505.02438,
// Sec. 2.3, Algorithm 1): the clamped, damped update of the design variables
// and the bisection on the multiplier lambda of the volume constraint.
//
// Bisection on the device.  A pass of k_oc_eval evaluates vol at the 15 nodes
// of the depth-4 tree of midpoints that the next 4 steps of the sequential
// loop can reach from the current bracket (l1, l2): node 0 is (l1 + l2) / 2,
// the child taken when vol > V* (l1 = mid) is 2k + 1, the other child
// (l2 = mid) is 2k + 2, each midpoint computed as the loop computes it.  Then
// k_oc_decide (one block) sums the block partials in a fixed order and walks
// the tree with the loop's test before every step, so it takes exactly the
// loop's decisions for this vol.  The state lives in device memory:
//   st[0] l1, st[1] l2, st[2] last mid, st[3] vol at it, st[4] steps,
//   st[5] done flag, st[6] max change.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"
#include "kernels.h"

namespace soptx {

namespace {

struct OcArgs {
    const double *rho, *dc, *dv;
    int64_t n;
    double move, eta;
    // the bisection's parameters (k_oc_search, k_oc_check, k_oc_finish)
    double target, lmax, tol;
    int max_steps;
};

// rho_new at lambda; comparisons written out so that a NaN propagates as it
// does through max / min of IEEE arithmetic with NaN operands
__device__ __forceinline__ double oc_new(double rho, double dc, double dv, double lam, double move, double eta) {
    const double num = -dc > 0.0 ? -dc : 0.0;
    const double B = num / (lam * dv);
    double be;
    if (eta == 0.5) be = sqrt(B);
    else if (eta == 1.0) be = B;
    else be = pow(B, eta);
    double c = rho * be;
    const double lo = rho - move > 0.0 ? rho - move : 0.0;
    const double hi = rho + move < 1.0 ? rho + move : 1.0;
    if (c < lo) c = lo;
    if (c > hi) c = hi;
    return c;
}

__device__ __forceinline__ void tree_mids(double l1, double l2, double (&lam)[kOcNodes]) {
    double a[kOcNodes], b[kOcNodes];
    a[0] = l1;
    b[0] = l2;
#pragma unroll
    for (int k = 0; k < kOcNodes; k++) {
        lam[k] = 0.5 * (a[k] + b[k]);
        if (2 * k + 2 < kOcNodes) {
            a[2 * k + 1] = lam[k];  // vol > V*: l1 = mid
            b[2 * k + 1] = b[k];
            a[2 * k + 2] = a[k];    // otherwise: l2 = mid
            b[2 * k + 2] = lam[k];
        }
    }
}

__global__ __launch_bounds__(256) void k_oc_init(double *st, double lmax, double *acc) {
    for (int x = threadIdx.x; x < kOcAcc; x += 256) acc[x] = 0.0;
    if (threadIdx.x < kOcSlots) st[8 + threadIdx.x] = 0.0;
    if (threadIdx.x == 0) {
        st[0] = 0.0;
        st[1] = lmax;
        st[2] = 0.0;
        st[3] = 0.0;
        st[4] = 0.0;
        st[5] = 0.0;
        st[6] = 0.0;
        st[7] = 0.0;
    }
}

// sum over the 64 lanes of a wave by a fixed butterfly (every lane gets it)
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// part[node * gridDim.x + block] = sum over the block's elements of dv rho_new(lambda_node):
// per thread in element order (by fma, as k_oc_check adds them: its volumes are
// these, bit for bit), then each wave by a butterfly, then the 4 waves in order
__global__ __launch_bounds__(256) void k_oc_eval(OcArgs A, const double *__restrict__ st, double *__restrict__ part) {
    __shared__ double red[4][kOcNodes];
    if (st[5] != 0.0) return;  // uniform: the bisection has ended
    double lam[kOcNodes], acc[kOcNodes];
    tree_mids(st[0], st[1], lam);
#pragma unroll
    for (int k = 0; k < kOcNodes; k++) acc[k] = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < A.n; e += (int64_t)gridDim.x * 256) {
        const double r = A.rho[e], d = A.dc[e], v = A.dv[e];
#pragma unroll
        for (int k = 0; k < kOcNodes; k++) acc[k] = fma(v, oc_new(r, d, v, lam[k], A.move, A.eta), acc[k]);
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kOcNodes; k++) {
        const double s = wave_sum(acc[k]);
        if (lane == 0) red[w][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < kOcNodes) {
        const int k = threadIdx.x;
        part[(int64_t)k * gridDim.x + blockIdx.x] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
}

// one wave per tree node (kOcNodes <= 16 waves of the 1024-thread block):
// lane l sums blocks l, l + 64, ... in order, then a butterfly
static_assert(kOcNodes <= 16, "one wave per tree node in a 1024-thread block");
__global__ __launch_bounds__(1024) void k_oc_decide(const double *__restrict__ part, int nblk, double vol_target,
                                                    double tol, int max_steps, double *st) {
    __shared__ double vol[kOcNodes];
    if (st[5] != 0.0) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (w < kOcNodes) {
        double t = 0.0;
        for (int b = lane; b < nblk; b += 64) t += part[(int64_t)w * nblk + b];
        t = wave_sum(t);
        if (lane == 0) vol[w] = t;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double l1 = st[0], l2 = st[1], lam = st[2], vl = st[3];
    int steps = (int)st[4];
    int node = 0;
    for (int level = 0; level < kOcDepth; level++) {
        if (!(l2 - l1 > tol * (l1 + l2) && steps < max_steps)) break;
        const double mid = 0.5 * (l1 + l2);
        if (vol[node] > vol_target) {
            l1 = mid;
            node = 2 * node + 1;
        } else {
            l2 = mid;
            node = 2 * node + 2;
        }
        lam = mid;
        vl = vol[(node - 1) / 2];
        steps++;
    }
    st[0] = l1;
    st[1] = l2;
    st[2] = lam;
    st[3] = vl;
    st[4] = (double)steps;
    st[5] = (l2 - l1 > tol * (l1 + l2) && steps < max_steps) ? 0.0 : 1.0;
}

// rho_new at the final multiplier, and block maxima of |rho_new - rho|
__global__ __launch_bounds__(256) void k_oc_apply(OcArgs A, const double *__restrict__ st, double *__restrict__ out,
                                                  double *__restrict__ part) {
    __shared__ double red[256];
    const double lam = st[2];
    double m = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < A.n; e += (int64_t)gridDim.x * 256) {
        const double r = A.rho[e];
        const double c = oc_new(r, A.dc[e], A.dv[e], lam, A.move, A.eta);
        out[e] = c;
        const double d = fabs(c - r);
        m = d > m || d != d ? d : m;
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            const double o = red[threadIdx.x + s];
            if (o > red[threadIdx.x] || o != o) red[threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_oc_change(const double *__restrict__ part, int nblk, double *st) {
    __shared__ double red[256];
    double m = 0.0;
    for (int b = threadIdx.x; b < nblk; b += 256) {
        const double o = part[b];
        if (o > m || o != o) m = o;
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            const double o = red[threadIdx.x + s];
            if (o > red[threadIdx.x] || o != o) red[threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) st[6] = red[0];
}

// ---- The same bisection, its path predicted and then proved (eta 0.5 and 1).
//
// With these exponents every operation of rho_new(lambda) is correctly
// rounded, hence monotone, and so are the products and the fixed-order sum:
// the vol that k_oc_eval computes is non-increasing in lambda, bit for bit.
// So three of its values decide every step of the sequential loop: if vol > V*
// at the path's last l1 and vol <= V* at its last l2, each midpoint that went
// up lies at or below that l1, each that went down at or above that l2, and
// the loop would have decided the same.  (vol at the path's first l1 has to be
// > V* as well: at a smaller lambda an overflow could still make a NaN.)  The
// one term that can rise with lambda, dv < 0 with rho < 0 and eta 1 (with eta
// 0.5 it is the root of a negative number), is a NaN in the proof, which fails.
//
// k_oc_search finds the root first: rho_new ~ clamp(s_e t) with s_e = rho
// sqrt(-dc / dv) and t = lambda^-1/2 (eta 1: rho (-dc) / dv and 1 / lambda)
// takes four operations a point instead of a divide and a square root, so a
// launch evaluates 63 multipliers: the octaves that max_steps halvings of lmax
// can reach, then twice the interval that holds the root.  These sums are in
// no fixed order (atomics, on one of 16 copies by block: 250 blocks on the same
// 63 addresses took 12 us): they only predict.  k_oc_check replays the
// loop's steps against the predicted root and evaluates vol at the three
// multipliers in k_oc_eval's order; k_oc_finish sums them in k_oc_decide's
// order and, if they prove the path, writes rho_new and the result.  If not
// (a sum within rounding of V* at a step, a NaN), nothing is written, and the
// passes above run.
// 192,000 elements, 37 steps: 3 searches of 7.5 us, the proof 9 and the finish
// 5 us with one host read, against 10 passes (12 launched) of 10.9 + 5.4 us
// with three; the call with the filter before it 102 against 342 us, and 121
// against 307 on 15,000 elements.  A search is bound by its chain (elements in,
// the sums so far, 63 points, one atomic a block); one point after the other
// instead of nine together took 11.4 us.

// sums of a wave's 64 floats, N at a time (lane 63 gets them): four shifts
// within rows of 16, then the row sums passed on
template <int N>
__device__ __forceinline__ void wave_sums_f32(float (&v)[N]) {
#define SOPTX_DPP(ctrl, rows)                                                                             \
    _Pragma("unroll") for (int j = 0; j < N; j++) v[j] +=                                                 \
        __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), ctrl, rows, 0xf, true))
    SOPTX_DPP(0x111, 0xf);
    SOPTX_DPP(0x112, 0xf);
    SOPTX_DPP(0x114, 0xf);
    SOPTX_DPP(0x118, 0xf);
    SOPTX_DPP(0x142, 0xa);
    SOPTX_DPP(0x143, 0xc);
#undef SOPTX_DPP
}

__device__ __forceinline__ double oc_scale(double lam, double eta) { return eta == 0.5 ? 1.0 / sqrt(lam) : 1.0 / lam; }

// The interval that holds the root, from b down L octaves; lane k of a wave
// stands for the search's point 2^(-(k + 1) L / 64) b, whose fraction of an
// octave is taken in FP32 (every kernel forms the same points; no kernel needs
// them closer).  va, vb: vol at the ends (negative: not known).
struct OcBracket {
    double b, va, vb;
    float L;
};
__device__ __forceinline__ double oc_point(const OcBracket &B, int k) {
    const float p = -(float)(k + 1) * (1.0f / 64.0f) * B.L;
    const float n = floorf(p);
    return ldexp(B.b * (double)__builtin_amdgcn_exp2f(p - n), (int)n);
}
// The sums of `done` searches ([search][copy][64] in acc) into LDS, by a block.
__device__ __forceinline__ void oc_sums(const double *acc, int done, double (&sum)[kOcSearch][4][64]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int p = 0; p < done; p++) {
        double t = 0.0;
#pragma unroll
        for (int c = 0; c < kOcCopies / 4; c++) t += acc[(p * kOcCopies + 4 * c + w) * 64 + lane];
        sum[p][w][lane] = t;
    }
    __syncthreads();
}
__device__ __forceinline__ OcBracket oc_bracket(const OcArgs &A, const double (&sum)[kOcSearch][4][64], int done,
                                                int lane) {
    OcBracket B;
    B.b = A.lmax;
    B.L = (float)(A.max_steps + 1);
    B.va = B.vb = -1.0;
    const int k = lane < kOcPoints ? lane : kOcPoints - 1;
    for (int p = 0; p < done; p++) {
        const double x = oc_point(B, k);
        const double v = (sum[p][0][k] + sum[p][1][k]) + (sum[p][2][k] + sum[p][3][k]);
        const unsigned long long m = __ballot(v > A.target);
        const int hit = m ? __ffsll((unsigned long long)m) - 1 : kOcPoints;
        if (hit > 0) {
            B.b = __shfl(x, hit - 1);
            B.vb = __shfl(v, hit - 1);
        }
        if (hit < kOcPoints) B.va = __shfl(v, hit);
        B.L *= 1.0f / 64.0f;
    }
    return B;
}

// elements of a thread at a time
constexpr int kOcEach = 3;

__global__ __launch_bounds__(256) void k_oc_search(OcArgs A, int done, double *__restrict__ acc) {
    __shared__ double scale[kOcPoints + 1];
    __shared__ float red[4][kOcPoints + 1];
    __shared__ double sum[kOcSearch][4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t e0 = (int64_t)blockIdx.x * (256 * kOcEach) + threadIdx.x;
    double s[kOcEach], lo[kOcEach], hi[kOcEach], dv[kOcEach];
    double r[kOcEach], d[kOcEach];
#pragma unroll
    for (int h = 0; h < kOcEach; h++) {
        const int64_t e = e0 + 256 * h;
        const bool ok = e < A.n;
        r[h] = ok ? A.rho[e] : 0.0;
        d[h] = ok ? A.dc[e] : 0.0;
        dv[h] = ok ? A.dv[e] : 0.0;
    }
    oc_sums(acc, done, sum);
    if (w == 0) {
        const OcBracket B = oc_bracket(A, sum, done, lane);
        scale[lane] = oc_scale(oc_point(B, lane), A.eta);
    }
#pragma unroll
    for (int h = 0; h < kOcEach; h++) {
        const double q = d[h] < 0.0 ? -d[h] / dv[h] : 0.0;
        s[h] = r[h] * (A.eta == 0.5 ? sqrt(q) : q);
        lo[h] = r[h] - A.move > 0.0 ? r[h] - A.move : 0.0;
        hi[h] = r[h] + A.move < 1.0 ? r[h] + A.move : 1.0;
    }
    __syncthreads();
    // nine points at a time, so that their sums' dependent steps overlap; lane k
    // keeps the wave's sum of point k
    constexpr int kBatch = 9;
    static_assert(kOcPoints % kBatch == 0, "whole batches");
    int mine = 0;
    for (int k0 = 0; k0 < kOcPoints; k0 += kBatch) {
        float f[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; j++) {
            const double t = scale[k0 + j];
            double x = 0.0;
#pragma unroll
            for (int h = 0; h < kOcEach; h++) x += dv[h] * fmin(fmax(s[h] * t, lo[h]), hi[h]);
            f[j] = (float)x;
        }
        wave_sums_f32(f);
#pragma unroll
        for (int j = 0; j < kBatch; j++) {
            const int v = __builtin_amdgcn_readlane(__float_as_int(f[j]), 63);
            mine = lane == k0 + j ? v : mine;
        }
    }
    red[w][lane] = __int_as_float(mine);
    __syncthreads();
    if (threadIdx.x < kOcPoints) {
        const int k = threadIdx.x;
        unsafeAtomicAdd(acc + (done * kOcCopies + blockIdx.x % kOcCopies) * 64 + k,
                        ((double)red[0][k] + (double)red[1][k]) + ((double)red[2][k] + (double)red[3][k]));
    }
}

// The loop's steps against the predicted root, by every block; block 0 leaves
// the path's end in st: [0] l1, [1] l2, [2] last midpoint, [4] steps, and which
// of the three values it is in [7].  Then vol at l1, l2 and the first l1.
__global__ __launch_bounds__(256) void k_oc_check(OcArgs A, const double *__restrict__ acc, double *__restrict__ st,
                                                  double *__restrict__ part) {
    __shared__ double lam[kOcProof];
    __shared__ double red[4][kOcProof];
    __shared__ double sum[kOcSearch][4][64];
    const int64_t e0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double r = 0.0, d = 0.0, v = 0.0;  // the thread's first element, read ahead of the sums
    if (e0 < A.n) {
        r = A.rho[e0];
        d = A.dc[e0];
        v = A.dv[e0];
    }
    oc_sums(acc, kOcSearch, sum);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (w == 0) {
        const OcBracket B = oc_bracket(A, sum, kOcSearch, lane);
        const double a = oc_point(B, 63);
        double root = 0.5 * (a + B.b);
        if (B.va > B.vb && B.vb >= 0.0) {
            const double ta = oc_scale(a, A.eta), tb = oc_scale(B.b, A.eta);
            const double t = tb + (A.target - B.vb) / (B.va - B.vb) * (ta - tb);
            root = A.eta == 0.5 ? 1.0 / (t * t) : 1.0 / t;
        }
        double l1 = 0.0, l2 = A.lmax, first = 0.0, mid = 0.0;
        int steps = 0;
        bool up = false;
        while (l2 - l1 > A.tol * (l1 + l2) && steps < A.max_steps) {
            mid = 0.5 * (l1 + l2);
            up = mid < root;
            if (up) {
                if (first == 0.0) first = mid;
                l1 = mid;
            } else {
                l2 = mid;
            }
            steps++;
        }
        if (lane == 0) {
            lam[0] = l1;
            lam[1] = l2;
            lam[2] = first;
            if (blockIdx.x == 0) {
                st[0] = l1;
                st[1] = l2;
                st[2] = mid;
                st[4] = (double)steps;
                st[7] = up ? 0.0 : 1.0;
            }
        }
    }
    __syncthreads();
    double a[kOcProof], l[kOcProof];
#pragma unroll
    for (int k = 0; k < kOcProof; k++) {
        a[k] = 0.0;
        l[k] = lam[k];
    }
    for (int64_t e = e0; e < A.n; e += (int64_t)gridDim.x * 256) {
        if (e != e0) {
            r = A.rho[e];
            d = A.dc[e];
            v = A.dv[e];
        }
#pragma unroll
        for (int k = 0; k < kOcProof; k++) a[k] = fma(v, oc_new(r, d, v, l[k], A.move, A.eta), a[k]);
        if (v < 0.0 && r < 0.0)
#pragma unroll
            for (int k = 0; k < kOcProof; k++) a[k] = __builtin_nan("");
    }
#pragma unroll
    for (int k = 0; k < kOcProof; k++) {
        const double s = wave_sum(a[k]);
        if (lane == 0) red[w][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < kOcProof) {
        const int k = threadIdx.x;
        part[(int64_t)k * gridDim.x + blockIdx.x] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
}

// Proof of the path, rho_new at its last midpoint and the largest change (as
// the bits of a non-negative double, whose order is its value's, a NaN above
// all).  nblk: blocks of k_oc_check.
__global__ __launch_bounds__(256) void k_oc_finish(OcArgs A, const double *__restrict__ part, int nblk, double *st,
                                                   double *__restrict__ out) {
    __shared__ double vol[4];
    __shared__ double red[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // the thread's first element, read ahead of the sums
    const int64_t e0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double r = 0.0, dc = 0.0, dv = 0.0;
    if (e0 < A.n) {
        r = A.rho[e0];
        dc = A.dc[e0];
        dv = A.dv[e0];
    }
    if (w < kOcProof) {
        // every load first, then the sum in k_oc_decide's order
        double x[kOcMaxBlocks / 64];
#pragma unroll
        for (int j = 0; j < kOcMaxBlocks / 64; j++)
            x[j] = lane + 64 * j < nblk ? part[(int64_t)w * nblk + lane + 64 * j] : 0.0;
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < kOcMaxBlocks / 64; j++)
            if (lane + 64 * j < nblk) t += x[j];
        t = wave_sum(t);
        if (lane == 0) vol[w] = t;
    }
    __syncthreads();
    const double l1 = st[0], l2 = st[1], lam = st[2];
    const bool low = l1 == 0.0 || (vol[0] > A.target && vol[2] > A.target);
    const bool high = l2 == A.lmax || vol[1] <= A.target;
    if (!(low && high)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st[3] = vol[st[7] == 0.0 ? 0 : 1];
        st[5] = 1.0;
    }
    double m = 0.0;
    for (int64_t e = e0; e < A.n; e += (int64_t)gridDim.x * 256) {
        if (e != e0) {
            r = A.rho[e];
            dc = A.dc[e];
            dv = A.dv[e];
        }
        const double c = oc_new(r, dc, dv, lam, A.move, A.eta);
        out[e] = c;
        const double d = fabs(c - r);
        m = d > m || d != d ? d : m;
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const double o = __shfl_xor(m, s);
        if (o > m || o != o) m = o;
    }
    if (lane == 0) red[w] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; k++)
            if (red[k] > m || red[k] != red[k]) m = red[k];
        atomicMax(reinterpret_cast<unsigned long long *>(st + 8 + blockIdx.x % kOcSlots),
                  (unsigned long long)__double_as_longlong(m));
    }
}

}  // namespace

int oc_blocks(int64_t n) {
    const int64_t b = (n + 255) / 256;
    return (int)(b < kOcMaxBlocks ? (b > 0 ? b : 1) : kOcMaxBlocks);
}

hipError_t launch_oc_init(double *st, double lmax, double *acc, hipStream_t s) {
    hipLaunchKernelGGL(k_oc_init, dim3(1), dim3(256), 0, s, st, lmax, acc);
    return hipGetLastError();
}

hipError_t launch_oc_direct(const double *rho, const double *dc, const double *dv, int64_t n, double move, double eta,
                            double vol_target, double lmax, double tol, int max_steps, double *st, double *acc,
                            double *part, double *out, hipStream_t s) {
    const OcArgs A{rho, dc, dv, n, move, eta, vol_target, lmax, tol, max_steps};
    const int g = oc_blocks(n);
    const unsigned gs = (unsigned)((n + 256 * kOcEach - 1) / (256 * kOcEach));
    hipError_t e;
    for (int p = 0; p < kOcSearch; p++) {
        hipLaunchKernelGGL(k_oc_search, dim3(gs), dim3(256), 0, s, A, p, acc);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_oc_check, dim3(g), dim3(256), 0, s, A, acc, st, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_oc_finish, dim3(g), dim3(256), 0, s, A, part, g, st, out);
    return hipGetLastError();
}

hipError_t launch_oc_pass(const double *rho, const double *dc, const double *dv, int64_t n, double move, double eta,
                          double vol_target, double tol, int max_steps, double *st, double *part, hipStream_t s) {
    const int g = oc_blocks(n);
    const OcArgs A{rho, dc, dv, n, move, eta, 0.0, 0.0, 0.0, 0};
    hipLaunchKernelGGL(k_oc_eval, dim3(g), dim3(256), 0, s, A, st, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_oc_decide, dim3(1), dim3(1024), 0, s, part, g, vol_target, tol, max_steps, st);
    return hipGetLastError();
}

hipError_t launch_oc_apply(const double *rho, const double *dc, const double *dv, int64_t n, double move, double eta,
                           double *st, double *out, double *part, hipStream_t s) {
    const int g = oc_blocks(n);
    const OcArgs A{rho, dc, dv, n, move, eta, 0.0, 0.0, 0.0, 0};
    hipLaunchKernelGGL(k_oc_apply, dim3(g), dim3(256), 0, s, A, st, out, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_oc_change, dim3(1), dim3(256), 0, s, part, g, st);
    return hipGetLastError();
}

}  // namespace soptx
