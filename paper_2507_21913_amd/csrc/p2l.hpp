// P2L (X list) of rows without reaction terms: the sources of a coarse leaf straight into the local of a
// finer box (log kernel; image rows for the Dirichlet and Neumann conditions, whose images carry a sign).
//
// LP lanes hold one X box's coefficients in registers and take its source rows r, r + LP, ...; per row
// and coefficient a complex multiply steps the power of sigma = rho / (z_j - c_b) and two multiply-adds
// per charge vector add it.  The factorials, signs of the kernel and 1/4pi are applied once at the end;
// the partial sums meet by lane moves, and lane s of a group adds coefficients s, s + LP, ... to the
// locals.  The rows come from a stream of sorted point indices per box (upper rows first), the index two
// steps and the point one step ahead of their use.  The boxes of 64 neighbours on a level are sorted by
// their rows, so that few lanes of a wave wait for its longest list.  The logarithm's imaginary part is
// not formed: in phi = H + conj(G) (G = H here; 2 Re H for a real impedance) it cancels, and no
// derivative contains lambda_0.
//
// Dipole sources (DIP) take the derivative along the source normal: the log local is holomorphic in
// d = z_j - c_b (upper box) or in conj(z_j) - c_b (image), so it is nu d/dd with nu = n_x + i n_y, or its
// conjugate for the image.
//
// What bounds it: the reads of scattered points and the read-modify-write of the locals: 450 MB in 175 us for
// the deep launch of the 4M curve, whose waves wait 73% of their time; issue (6 (p + 1) FP64 operations per
// row and ~80 for its geometry) is 27% there, and 48% with eight vectors on the 2M forest.  Two vectors
// share the powers up to p = 20; beyond, their sums would not leave two waves per SIMD.  At p = 15 with
// sixteen lanes a box, one vector's sums spill 8 registers (10 for dipoles) of the 128 of four waves.
// The kernel it replaced formed the terms of 64 rows in LDS and summed them from there, at seven waves per
// CU.  All launches of an evaluation alone on the GPU: 4M points along a curve, p = 30: 1,035 -> 255 us;
// 2M points in 64 instances, p = 20, eight vectors: 1,205 -> 367 us (and 33 us for the rows with reaction
// terms).
#pragma once
#include "internal.hpp"
#include "special.hpp"

namespace fmmhp {

// Lane moves within a wave by DPP (no LDS traffic, a few cycles), for doubles as two 32-bit halves.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Lane l's value of x in every lane (l uniform; reads the lane's register whatever the exec mask).
__device__ __forceinline__ double read_lane_f64(double x, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
    return __hiloint2double(hi, lo);
}

// Sum over aligned groups of IA = 1, 2, 4, 8 or 16 consecutive lanes (every lane of a group gets it).
__device__ __forceinline__ double lane_group_sum(double s, int IA) {
    if (IA >= 2) s += dpp_move<0xB1, 0xF>(s);   // quad_perm [1, 0, 3, 2]
    if (IA >= 4) s += dpp_move<0x4E, 0xF>(s);   // quad_perm [2, 3, 0, 1]
    if (IA >= 8) s += dpp_move<0x141, 0xF>(s);  // row_half_mirror
    if (IA >= 16) s += dpp_move<0x140, 0xF>(s);  // row_mirror
    return s;
}

constexpr int kP2LChunk = 64;  // X boxes sorted by their rows together

struct P2LArgs {
    int nslot, nbox, nloc, nv;
    const int4 *slot;        // {box, rows, upper rows, 0}
    const int64_t *row0;     // first row of each slot in the stream
    const double4 *geo;      // {centre x, centre y, half side, instance} of each slot
    const int32_t *stream;   // sorted point indices
    const double2 *xy, *nrm;
    const double *qs;        // [n][nv]
    const double *logside, *fact;
    double isg;              // sign of an image's log kernel
    cplx *Lam;
};

__host__ __device__ constexpr int p2l_vecs(int PB, int NV) { return NV % 2 == 0 && PB <= 20 ? 2 : 1; }

// The stream's rows of one list entry {leaf, 0, row (low, high)}.
__global__ void k_p2l_rows(int64_t m, const int4 *__restrict__ ent, const int32_t *__restrict__ first,
                           const int32_t *__restrict__ count, int32_t *__restrict__ stream) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m) return;
    const int4 en = ent[e];
    int32_t *dst = stream + ((int64_t)en.w << 32 | (uint32_t)en.z);
    const int f = first[en.x], n = count[en.x];
    for (int i = 0; i < n; ++i) dst[i] = f + i;
}

template <int VP, bool DIP>
struct P2LRow {
    double2 z, nu;
    double q[VP];
    __device__ __forceinline__ void load(const P2LArgs &a, int j, int v0) {
        z = a.xy[j];
        if (DIP) nu = a.nrm[j];
        if constexpr (VP == 2) {
            const double2 t = *(const double2 *)(a.qs + (int64_t)j * a.nv + v0);  // v0 and nv are even
            q[0] = t.x;
            q[1] = t.y;
        } else {
            q[0] = a.qs[(int64_t)j * a.nv + v0];
        }
    }
};

template <int PB, bool DIP, int VP, int LP>
__global__ __launch_bounds__(256, VP == 2 ? (PB <= 5 ? 4 : PB <= 10 ? 3 : 2) : PB <= 15 ? 4 : PB <= 20 ? 3 : 2) void k_p2l(P2LArgs a) {
    constexpr int P1 = PB + 1;
    // an XCD takes one contiguous run of chunks: neighbouring boxes share lines of the locals
    const int per = gridDim.x / 8;
    const int c = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    const int v0 = blockIdx.y * VP;
    const int sub = threadIdx.x & (LP - 1);
    const int s = c * (256 / LP) + threadIdx.x / LP;
    const bool have = s < a.nslot;
    const int4 sl = have ? a.slot[s] : make_int4(0, 0, 0, 0);
    const int64_t r0 = have ? a.row0[s] : 0;
    const double4 g = have ? a.geo[s] : make_double4(0.0, 0.0, 1.0, 0.0);
    const double irho = 1.0 / g.z;
    const double lrho = DIP ? 0.0 : a.logside[sl.x] - (kLn2Hi + kLn2Lo);
    const int32_t *st = a.stream + r0;
    const int K = sl.y;
    cplx acc[VP][P1];
#pragma unroll
    for (int v = 0; v < VP; ++v)
#pragma unroll
        for (int m = 0; m < P1; ++m) acc[v][m] = mk(0.0, 0.0);
    int j1 = sub + LP < K ? st[sub + LP] : 0;
    P2LRow<VP, DIP> nx;
    if (sub < K) nx.load(a, st[sub], v0);
    for (int r = sub; r < K; r += LP) {
        const P2LRow<VP, DIP> cu = nx;
        nx.load(a, j1, v0);  // (point 0 past the end)
        j1 = r + 2 * LP < K ? st[r + 2 * LP] : 0;
        const bool img = r >= sl.z;
        const double dx = (cu.z.x - g.x) * irho, dy = ((img ? -cu.z.y : cu.z.y) - g.y) * irho;
        const double r2 = fma(dx, dx, dy * dy);
        const double ir = 1.0 / r2;
        const cplx sig = mk(dx * ir, -(dy * ir));
        const double sg = img ? -a.isg : 1.0;
        cplx pw = sig;
        if (DIP) pw = mk(cu.nu.x, img ? -cu.nu.y : cu.nu.y) * sig;
        double q[VP];
#pragma unroll
        for (int v = 0; v < VP; ++v) q[v] = sg * cu.q[v];
        if (!DIP) {
            const double lg = fma(0.5, log(r2), lrho);
#pragma unroll
            for (int v = 0; v < VP; ++v) acc[v][0].re = fma(-q[v], lg, acc[v][0].re);
        }
#pragma unroll
        for (int m = DIP ? 0 : 1; m < P1; ++m) {
#pragma unroll
            for (int v = 0; v < VP; ++v) {
                acc[v][m].re = fma(q[v], pw.re, acc[v][m].re);
                acc[v][m].im = fma(q[v], pw.im, acc[v][m].im);
            }
            if (m < PB) pw = pw * sig;
        }
    }
#pragma unroll
    for (int v = 0; v < VP; ++v) {
        // log: lambda_m += (m - 1)!/(4 pi) acc_m;  dipoles: lambda_m -= m!/(4 pi rho) acc_m
        const double sc = DIP ? -kInv4Pi * irho : kInv4Pi;
#pragma unroll
        for (int i = 0; i < (P1 + LP - 1) / LP; ++i) {
            const int m = LP * i + sub;
            cplx t = mk(0.0, 0.0);
#pragma unroll
            for (int k = 0; k < LP; ++k)
                if (LP * i + k < P1) {
                    const double re = lane_group_sum(acc[v][LP * i + k].re, LP);
                    const double im = lane_group_sum(acc[v][LP * i + k].im, LP);
                    t.re = sub == k ? re : t.re;
                    t.im = sub == k ? im : t.im;
                }
            if (m < P1 && K > 0) {
                const double f = sc * a.fact[DIP ? m : m > 0 ? m - 1 : 0];
                for (int ld = 0; ld < a.nloc; ++ld) {
                    cplx *dst = a.Lam + (((int64_t)(v0 + v) * a.nloc + ld) * P1 + m) * a.nbox + sl.x;
                    cplx o = *dst;
                    o.re = fma(f, t.re, o.re);
                    o.im = fma(f, t.im, o.im);
                    *dst = o;
                }
            }
        }
    }
}

}  // namespace fmmhp
