// M2L of upper sources through plane waves.
//
// In units of the half side rho, an upper source box at offset zeta = 2 (dx + i dy) contributes
//   lambda_n += (1/4pi) sum_m (n+m-1)!/zeta^(n+m) w_m      (n + m >= 1; L w_0 for n = m = 0),
// a Hankel contraction of 4 (p+1)^2 real multiply-adds per pair.  For Re zeta > 0,
// (j-1)!/zeta^j = int_0^inf mu^(j-1) e^(-mu zeta) dmu, and a quadrature {mu_k, omega_k} of this integral
// makes the translation diagonal (Hrycak and Rokhlin, "An improved fast multipole algorithm for
// potential fields", 1998):
//   X_E = sum_m mu_k^m w_m (per source box),  lambda_n += sum_k (omega_k/(4pi mu_k)) mu_k^n e^(-mu_k zeta) X_E,
// with i^n-rotated sums for the north, west and south directions.  N and S take the rows |dy| >= 2 of
// the 6 x 6 block around a parent, E and W the rest.  The four directions of a box come from the four
// sums of its coefficients m = r (mod 4), and the same the other way round, so that each end costs
// 2 (p+1) multiply-adds per node instead of one Hankel row per pair: at p = 20, 34 nodes and 27 pairs
// per box the whole translation takes ~9 K operations per box against 47.6 K.
// The n = m = 0 term of the quadrature is taken out again exactly: it is a constant per offset times
// w_0, folded with the logarithm into the table Lp.
//
// One workgroup per tile: up to 32 parents of one level (their children are the targets) whose upper
// colleagues number at most kPwCells (their children are the sources).  Waves 0-3 are the source
// waves: wave q holds the multipoles of the tile's source children in quadrant q in registers, one
// box per lane, and writes the four outgoing waves of the step's two nodes to LDS.  Waves 4-7 are the
// target waves: wave 4 + by + 2 par takes the children in row by of the 32 parents (lane = (parent,
// bx)) at the nodes of parity par, sums the incoming waves and holds the locals in registers.  The two
// sides run one step apart on double-buffered LDS with one barrier per step.  What bounds it: the
// latency of a step (scalar loads, LDS reads, lane swaps, barrier), which the second workgroup on the CU
// covers in part.  By the counters (1M points, p = 20; 4M curve, p = 30; each launch alone) its waves wait
// 53-61% of their time and the vector instructions take 31% of it, the LDS reads with their bank conflicts
// (4.6 cycles a read) about as much; 120 MB of HBM traffic at 1M, twice the boxes' expansions.  The lanes bx = 0, 1 of
// a parent share their sums: each takes the three nearest columns on its own side and the partner's
// half comes by a lane swap; what differs between the lanes and between the two rows is a sign, so
// all four child positions run the same code.  A cell without a source box reads a zero column, so a
// box's result does not depend on the tile it is in.
//
// Measured, all launches of an evaluation alone on the GPU, against the Hankel rows of k_m2l: 1M uniform
// points, p = 20, leaf 32: 359 -> 80 us; 4M points along a curve, p = 30, leaf 40: 1,407 -> 398 us;
// 2M points in 64 instances, p = 20, eight vectors: 3,790 -> 855 us; one tile (2,000 points): 90 -> 20 us.
// Potentials of random charges agree with the Hankel rows' to a few times err of pw_nodes.hpp, which also
// gives the quadrature's largest errors.
#pragma once
#include "internal.hpp"
#include "pw_nodes.hpp"

namespace fmmhp {

constexpr int kPwPar = 32;         // parents per tile (x 4 children = targets)
constexpr int kPwCells = 63;       // source parents per tile; cell 63 is the zero column
constexpr int kPwStride = 65;      // cells per LDS row (odd: the four quadrants fall on different banks)
constexpr int kPwConst = 9;        // constants of a node ahead of its g mu^n row

__host__ __device__ constexpr int pw_steps(int PB) { return (pw_nodes(PB) + 1) / 2; }
__host__ __device__ constexpr int pw_src_row(int PB) { return (PB + 8) / 8 * 8; }
__host__ __device__ constexpr int pw_tgt_row(int PB) { return (kPwConst + PB + 8) / 8 * 8; }

struct PwArgs {
    int nbox, tile0, nloc;
    const int32_t *src;      // [tiles][4][64] source boxes by quadrant, -1: none
    const int32_t *tgt;      // [tiles][4][kPwPar] target boxes by quadrant, -1: none
    const uint64_t *cells;   // [tiles][kPwPar] cell of each of a parent's eight colleagues (a byte each)
    const double *ts, *tt;   // node tables of the source and target waves
    const cplx *Lp;          // [kNumSlots]
    const double *logside;
    const cplx *W;
    cplx *Lam;
};

__device__ __forceinline__ double pw_swap(double v) {  // the value of lane ^ 1 (quad_perm [1, 0, 3, 2])
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xB1, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xB1, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// The node tables are read through the constant address space: the loads are then scalar (one value for
// the wave, into SGPRs); as plain global reads between barriers they came out as vector loads.
typedef __attribute__((address_space(4))) const double *pw_tab;
__device__ __forceinline__ pw_tab pw_const(const double *p) { return (pw_tab)(uintptr_t)p; }

// LDS index of (node of the step, direction, quadrant, cell); directions 0 E, 1 W, 2 N, 3 S.
__device__ __forceinline__ int pw_at(int node, int dir, int quad, int cell) {
    return ((node * 4 + dir) * 4 + quad) * kPwStride + cell;
}

constexpr int kPwBuf = 2 * 4 * 4 * kPwStride;  // complex values per LDS buffer

// The target side: row BY of the tile's children, the nodes of parity par (both uniform in the wave).
template <int PB, int BY>
__device__ __forceinline__ void pw_targets(const PwArgs &a, cplx *sX, const double *sW0, int tile, int par, int lane,
                                           int64_t vec) {
    constexpr int P1 = PB + 1, NS = pw_steps(PB), TT = pw_tgt_row(PB), H = (P1 + 1) / 2;
    constexpr int NY = 1 - BY;
    constexpr int tau = BY ? -1 : 1;  // +1: the far side of this row is north
    const int bx = lane & 1, nx = 1 - bx, pi = lane >> 1;
    const int b = a.tgt[((int64_t)tile * 4 + (bx | BY << 1)) * kPwPar + pi];
    const int sig = bx ? -1 : 1;      // +1: the lane's own side is east
    // far row F (two box rows), near row G (one), middle row M; own column, own side, opposite side
    int oF, sF, eF, oG, sG, pG, sM, pM;
    {
        // colleague bytes in the order (-1,-1) (0,-1) (1,-1) (-1,0) (1,0) (-1,1) (0,1) (1,1)
        const uint64_t cw = a.cells[(int64_t)tile * kPwPar + pi];
        auto cell = [&](int k) { return (int)((cw >> (8 * k)) & 255); };
        constexpr int rF = BY ? 0 : 5, rG = BY ? 5 : 0;
        oF = cell(rF + 1);
        sF = cell(rF + 1 + sig);
        eF = cell(rF + 1 - sig);
        oG = cell(rG + 1);
        sG = cell(rG + 1 + sig);
        pG = cell(rG + 1 - sig);
        sM = bx ? cell(3) : cell(4);
        pM = bx ? cell(4) : cell(3);
    }
    // LDS positions without the box row, which is added as a constant: columns 1/2, 3/2, 5/2 boxes from
    // the parent's centre on the own side; the east and west columns two boxes from the child
    constexpr int RN = 2 * BY * kPwStride, RY = 2 * NY * kPwStride;
    constexpr int DF = (BY ? 3 : 2) * 4 * kPwStride, DG = (BY ? 2 : 3) * 4 * kPwStride;
    const int p0 = par * 16 * kPwStride, dA = p0 + (bx ? 4 : 0) * kPwStride, dB = p0 + (bx ? 0 : 4) * kPwStride;
    const int qx = bx * kPwStride, qn = nx * kPwStride;
    const int f1 = p0 + qn + oF, f3 = p0 + qx + sF, f5 = p0 + qn + sF;
    const int g1 = p0 + qn + oG, g3 = p0 + qx + sG, g5 = p0 + qn + sG;
    const int aM = dA + qx + sM, aG = dA + qx + sG, bM = dB + qx + pM, bG = dB + qx + pG;
    const double dsig = (double)sig;
    cplx lam[P1];
#pragma unroll
    for (int n = 0; n < P1; ++n) lam[n] = mk(0.0, 0.0);
    __syncthreads();
    {
        // the logarithm: this wave's half of the 27 offsets (parity 0 the lane's own columns, parity
        // 1 the partner's, seen from this child: quadrant bits mirrored in x)
        const double ll = b >= 0 ? a.logside[b] * 0.07957747154594766788 : 0.0;
        auto add = [&](int dx, int dy, int row, int at) {
            const double w0 = sW0[row + at];
            const cplx L = a.Lp[(dy + 3) * 7 + dx + 3];
            lam[0].re = fma(L.re - ll, w0, lam[0].re);
            lam[0].im = fma(L.im, w0, lam[0].im);
        };
        const int fo = par ? qx + oF : qn + oF, go = par ? qx + oG : qn + oG;
        const int f3_ = par ? qn + eF : qx + sF, f5_ = par ? qx + eF : qn + sF;
        const int g3_ = par ? qn + pG : qx + sG, g5_ = par ? qx + pG : qn + sG;
        const int d1 = par ? 0 : sig, dd = par ? -sig : sig;
        add(d1, 2 * tau, RN, fo);
        add(d1, 3 * tau, RY, fo);
        add(d1, -2 * tau, RN, go);
        add(d1 + dd, 2 * tau, RN, f3_);
        add(d1 + dd, 3 * tau, RY, f3_);
        add(d1 + dd, -2 * tau, RN, g3_);
        add(d1 + 2 * dd, 2 * tau, RN, f5_);
        add(d1 + 2 * dd, 3 * tau, RY, f5_);
        add(d1 + 2 * dd, -2 * tau, RN, g5_);
        // own side: two boxes away (the lane's own column), three (the partner's opposite one)
        const int qs = par ? qn : qx, ds = par ? 3 * sig : 2 * sig;
        add(ds, 0, RN, qs + sM);
        add(ds, tau, RY, qs + sM);
        add(ds, -tau, RY, qs + sG);
        if (par == 0) {
            add(-2 * sig, 0, RN, qx + pM);
            add(-2 * sig, tau, RY, qx + pM);
            add(-2 * sig, -tau, RY, qx + pG);
        }
    }
#pragma unroll 1
    for (int j = 0; j < NS; ++j) {
        const pw_tab t = pw_const(a.tt + (2 * j + par) * TT);
        const cplx *X = sX + (j & 1) * kPwBuf;
        const double f = t[0], c1 = t[1], s1 = t[2], c3 = t[3], s3 = t[4], c5 = t[5], s5 = t[6], c2 = t[7], s2 = t[8];
        // a side's three columns: sum of x e^(+-i mu u), the partner's half, the shift to the child
        auto row = [&](cplx x1, cplx x3, cplx x5, double sg) {
            const double cr = fma(c5, x5.re, fma(c3, x3.re, c1 * x1.re)), ci = fma(c5, x5.im, fma(c3, x3.im, c1 * x1.im));
            const double dr = fma(s5, x5.re, fma(s3, x3.re, s1 * x1.re)), di = fma(s5, x5.im, fma(s3, x3.im, s1 * x1.im));
            double tr = fma(-sg, di, cr), ti = fma(sg, dr, ci);
            tr += pw_swap(tr);
            ti += pw_swap(ti);
            const double sh = sg * s1;
            return mk(fma(c1, tr, -(sh * ti)), fma(c1, ti, sh * tr));
        };
        auto two = [&](int at) {  // near row + e^(-2 mu) far row
            const cplx n_ = X[DF + RN + at], f_ = X[DF + RY + at];
            return mk(fma(f, f_.re, n_.re), fma(f, f_.im, n_.im));
        };
        const double dst = tau * dsig;
        const cplx F = row(two(f1), two(f3), two(f5), dst);
        if (PB > 10) __builtin_amdgcn_sched_barrier(0);
        const cplx G = row(X[DG + RN + g1], X[DG + RN + g3], X[DG + RN + g5], -dst);
        if (PB > 10) __builtin_amdgcn_sched_barrier(0);
        const double ss = dst * s2;
        auto col = [&](cplx x0, cplx xF, cplx xG, double sg) {  // x0 + c2 (xF + xG) + i sg (xF - xG)
            const cplx s = xF + xG, d = xF - xG;
            return mk(fma(c2, s.re, fma(-sg, d.im, x0.re)), fma(c2, s.im, fma(sg, d.re, x0.im)));
        };
        const cplx B = col(X[RN + bM], X[RY + bM], X[RY + bG], ss);
        const cplx Aa = col(X[RN + aM], X[RY + aM], X[RY + aG], -ss);
        const cplx U = mk(fma(f, pw_swap(B.re), Aa.re), fma(f, pw_swap(B.im), Aa.im));
        const cplx ewp = U + B, ewm = dsig * (U - B), nsp = F + G, nsm = (double)tau * (F - G);
        const cplx L[4] = {ewp + nsp, mk(ewm.re + nsm.im, ewm.im - nsm.re), ewp - nsp,
                           mk(ewm.re - nsm.im, ewm.im + nsm.re)};
        if (PB > 10) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < P1; ++n) {
            lam[n].re = fma(t[kPwConst + n], L[n & 3].re, lam[n].re);
            lam[n].im = fma(t[kPwConst + n], L[n & 3].im, lam[n].im);
        }
        __syncthreads();
    }
    // the two parities' halves: parity 0 finishes the coefficients below H, parity 1 the others
    cplx *ex = sX + BY * 64 * P1 + lane;
#pragma unroll
    for (int n = 0; n < P1; ++n)
        if ((n < H) == (par == 1)) ex[n * 64] = lam[n];
    __syncthreads();
    if (b < 0) return;
    cplx *Lam = a.Lam + vec * a.nloc + b;
    const int64_t second = (int64_t)P1 * a.nbox;
#pragma unroll
    for (int n = 0; n < P1; ++n)
        if ((n < H) == (par == 0)) {
            const cplx v = lam[n] + ex[n * 64];
            Lam[(int64_t)n * a.nbox] = v;
            if (a.nloc == 2) Lam[second + (int64_t)n * a.nbox] = v;
        }
}

// p <= 20: 128 registers, two workgroups (16 waves) per CU.  They do not quite hold p = 20: 14 spills, 52
// bytes of scratch a lane, two of them LDS addresses that one row's target waves reload in every step, the
// others before and after the steps (one spill at p = 10); two workgroups were still faster than one of 180
// registers (1M points: 99 -> 80 us with the scalar table loads).  Above, the locals alone take up to 164
// and one workgroup fits: 164, 194, 224 and 254 registers, no spills.
template <int PB>
__global__ __launch_bounds__(512, PB <= 20 ? 4 : 2) void k_m2l_pw(PwArgs a) {
    constexpr int P1 = PB + 1, NS = pw_steps(PB), TS = pw_src_row(PB);
    constexpr int NX = 2 * kPwBuf > 2 * 64 * P1 ? 2 * kPwBuf : 2 * 64 * P1;
    __shared__ cplx sX[NX];
    __shared__ double sW0[4 * kPwStride];
    const int tile = blockIdx.x + a.tile0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t vec = (int64_t)blockIdx.y * P1 * a.nbox;
    if (wave >= 4) {
        const int par = (wave >> 1) & 1;
        if (wave & 1) pw_targets<PB, 1>(a, sX, sW0, tile, par, lane, vec);
        else pw_targets<PB, 0>(a, sX, sW0, tile, par, lane, vec);
        return;
    }
    const int b = a.src[((int64_t)tile * 4 + wave) * 64 + lane];
    const cplx *W = a.W + vec + max(b, 0);
    cplx w[P1];
#pragma unroll
    for (int n = 0; n < P1; ++n) {
        w[n] = W[(int64_t)n * a.nbox];
        if (b < 0) w[n] = mk(0.0, 0.0);
    }
    sW0[wave * kPwStride + lane] = w[0].re;
    cplx *out = sX + wave * kPwStride + lane;
    // step j's waves go to buffer j mod 2 while the target waves read step j - 1's from the other
#pragma unroll 1
    for (int j = 0; j <= NS; ++j) {
        if (j < NS) {
            cplx *o = out + (j & 1) * kPwBuf;
#pragma unroll
            for (int node = 0; node < 2; ++node, o += 16 * kPwStride) {
                const pw_tab t = pw_const(a.ts + (2 * j + node) * TS);
                cplx A[4] = {w[0], mk(0.0, 0.0), mk(0.0, 0.0), mk(0.0, 0.0)};
#pragma unroll
                for (int n = 1; n < P1; ++n) {
                    A[n & 3].re = fma(t[n], w[n].re, A[n & 3].re);
                    A[n & 3].im = fma(t[n], w[n].im, A[n & 3].im);
                }
                const cplx P0 = A[0] + A[2], Q1 = A[1] + A[3], M0 = A[0] - A[2], M1 = A[1] - A[3];
                o[0] = P0 + Q1;                                         // E
                o[4 * kPwStride] = P0 - Q1;                             // W
                o[8 * kPwStride] = mk(M0.re + M1.im, M0.im - M1.re);    // N: M0 - i M1
                o[12 * kPwStride] = mk(M0.re - M1.im, M0.im + M1.re);   // S: M0 + i M1
            }
        }
        __syncthreads();
    }
    __syncthreads();
}

}  // namespace fmmhp
