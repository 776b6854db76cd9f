// M2M and L2L: bands of up to three levels per launch, expansions in registers.
//
// A lane holds the whole expansion of one box.  The shift of a child at eps = (+-1/2, +-1/2) (units of
// the parent's half side) is the Toeplitz product of eqs. (metome) / (truncatedL2L),
//   w^P_n = sum_{m<=n} (-eps)^(n-m)/(n-m)! 2^-m w^c_m,   lambda^c_m = 2^-m sum_{n>=m} eps^(n-m)/(n-m)! lambda^P_n,
// and eps^(n-m) = eps^n eps^-m: with the powers on either side the product in the middle is real,
// (p+1)(p+2)/2 pairs of multiply-adds with the same constants 1/k! for every lane, done in place.  The
// powers of +-1/2 +- i/2 have components 0 or +-2^-k and are exact.
//
// A band takes the levels root .. root + nlev (nlev <= 3).  A wave holds 4^(3 - nlev) roots; lane =
// (root, position at the deepest level, two bits per level), so that the lanes of one ancestor are
// neighbours.  Going up, the shifted expansions of four siblings meet by lane moves (in the order
// (0 + 1) + (2 + 3) whatever the band), and every lane of the parent goes on with the sum; a box that
// is a leaf itself brings its own.  Going down, every lane follows its own line of ancestors, adding
// each box's own local on the way.  Empty positions carry zeros; a level that is empty in the whole
// wave is skipped.
//
// What bounds it: a few thousand cycles of FP64 issue per level and wave, at two waves per SIMD up to p = 20
// and one from p = 30 (256 registers, and accumulation registers that hold the rest of x by copies: 2 and 56
// at p = 30, 90 and 160 at p = 40, M2M and L2L; the L2L has 8 at p = 25), behind one or two memory latencies
// per band.  The passes it replaced kept subtrees in LDS and were
// bound by LDS reads (two 16-byte reads per four multiply-adds) and one launch per level above.  Alone
// on the GPU, all launches of an evaluation: 1M uniform points, p = 20: M2M 98 -> 38 us, L2L 62 -> 39 us;
// 20,000 points along a curve (depth 10, complex impedance), p = 30: M2M 99 -> 49 us, L2L 188 -> 46 us;
// 4M along it (depth 15): M2M 450 -> 155 us, L2L 680 -> 245 us; 2M points in 64 instances, eight
// vectors: M2M 702 -> 196 us, L2L 398 -> 260 us.
#pragma once
#include "internal.hpp"

namespace fmmhp {

constexpr int32_t kBandNonLeaf = 1 << 30;  // flag of a box id in the band tables (ids stay below 2^28)

struct InvFact {
    double c[42];
    constexpr InvFact() : c() {
        double f = 1.0;
        for (int k = 0; k < 42; ++k) {
            c[k] = 1.0 / f;
            f *= k + 1;
        }
    }
};

// x_n *= s^n (s = (a, b), components +-1/2)
template <int P1>
__device__ __forceinline__ void band_rotate(cplx (&x)[P1], double a, double b) {
    double fr = 1.0, fi = 0.0;
#pragma unroll
    for (int n = 1; n < P1; ++n) {
        const double t = fma(fr, a, -(fi * b));
        fi = fma(fr, b, fi * a);
        fr = t;
        x[n] = mk(fma(fr, x[n].re, -(fi * x[n].im)), fma(fr, x[n].im, fi * x[n].re));
    }
}

// x_n <- sum_{m<=n} x_m/(n-m)!, in place from the highest n; four n at a time are independent chains,
// and the barriers keep the compiler from holding old and new values of more.  (Constant trip counts
// throughout: a loop that is not unrolled in full puts x into scratch memory.)
template <int P1>
__device__ __forceinline__ void band_toeplitz_up(cplx (&x)[P1]) {
    constexpr InvFact inv;
    constexpr int NG = (P1 + 2) / 4;  // groups of n: P1 - 1 .. 1
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int top = P1 - 1 - 4 * g;
        // inside the group from the top (its lower values are still the old ones), then from below it
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = i + 1; j < 4; ++j)
                if (top - j >= 0) {
                    x[top - i].re = fma(inv.c[j - i], x[top - j].re, x[top - i].re);
                    x[top - i].im = fma(inv.c[j - i], x[top - j].im, x[top - i].im);
                }
#pragma unroll
        for (int m = P1 - 1; m >= 0; --m)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (m <= top - 4) {
                    x[top - i].re = fma(inv.c[top - i - m], x[m].re, x[top - i].re);
                    x[top - i].im = fma(inv.c[top - i - m], x[m].im, x[top - i].im);
                }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// x_m <- sum_{n>=m} x_n/(n-m)!, in place from the lowest m.
template <int P1>
__device__ __forceinline__ void band_toeplitz_down(cplx (&x)[P1]) {
    constexpr InvFact inv;
    constexpr int NG = (P1 + 2) / 4;  // groups of m: 0 .. P1 - 2
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int bot = 4 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = i + 1; j < 4; ++j)
                if (bot + j < P1) {
                    x[bot + i].re = fma(inv.c[j - i], x[bot + j].re, x[bot + i].re);
                    x[bot + i].im = fma(inv.c[j - i], x[bot + j].im, x[bot + i].im);
                }
#pragma unroll
        for (int n = 0; n < P1; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (n >= bot + 4) {
                    x[bot + i].re = fma(inv.c[n - bot - i], x[n].re, x[bot + i].re);
                    x[bot + i].im = fma(inv.c[n - bot - i], x[n].im, x[bot + i].im);
                }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Sum over the four siblings at level k of the lane's position (all lanes below a sibling hold the same
// value).
__device__ __forceinline__ double band_dpp(double v, int which) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    switch (which) {
    case 0: lo = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xF, 0xF, false), hi = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xF, 0xF, false); break;   // lane ^ 1
    case 1: lo = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xF, 0xF, false), hi = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xF, 0xF, false); break;   // lane ^ 2
    case 2: lo = __builtin_amdgcn_update_dpp(0, lo, 0x141, 0xF, 0xF, false), hi = __builtin_amdgcn_update_dpp(0, hi, 0x141, 0xF, 0xF, false); break; // the other quad of 8 lanes
    default: lo = __builtin_amdgcn_update_dpp(0, lo, 0x140, 0xF, 0xF, false), hi = __builtin_amdgcn_update_dpp(0, hi, 0x140, 0xF, 0xF, false); break; // the other half of 16
    }
    return __hiloint2double(hi, lo);
}

template <int P1>
__device__ __forceinline__ void band_sum(cplx (&x)[P1], int k) {
    if (k == 2) {
#pragma unroll
        for (int n = 0; n < P1; ++n) {
            x[n].re += __shfl_xor(x[n].re, 16);
            x[n].im += __shfl_xor(x[n].im, 16);
        }
#pragma unroll
        for (int n = 0; n < P1; ++n) {
            x[n].re += __shfl_xor(x[n].re, 32);
            x[n].im += __shfl_xor(x[n].im, 32);
        }
    } else if (k == 1) {
#pragma unroll
        for (int n = 0; n < P1; ++n) {
            x[n].re += band_dpp(x[n].re, 2);
            x[n].im += band_dpp(x[n].im, 2);
            x[n].re += band_dpp(x[n].re, 3);
            x[n].im += band_dpp(x[n].im, 3);
        }
    } else {
#pragma unroll
        for (int n = 0; n < P1; ++n) {
            x[n].re += band_dpp(x[n].re, 0);
            x[n].im += band_dpp(x[n].im, 0);
            x[n].re += band_dpp(x[n].re, 1);
            x[n].im += band_dpp(x[n].im, 1);
        }
    }
}

// tab: [waves][nlev + 1][64] box (or -1) of each lane at the band's levels, deepest first.
template <int PB>
__global__ __launch_bounds__(256) void k_m2m_band(int nwave, int nlev, const int32_t *__restrict__ tab, int nbox,
                                                  cplx *__restrict__ W) {
    constexpr int P1 = PB + 1;
    __builtin_amdgcn_s_setprio(3);  // upward pass: the critical path
    const int wv = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (wv >= nwave) return;
    const int lane = threadIdx.x & 63;
    W += (int64_t)blockIdx.y * P1 * nbox;  // charge vector
    tab += (int64_t)wv * (nlev + 1) * 64 + lane;
    int id = tab[0];
    cplx x[P1];
    bool zero = __ballot(id >= 0) == 0;  // the wave holds nothing at this level
    {
        const cplx *w = W + (id >= 0 ? id & (kBandNonLeaf - 1) : 0);
#pragma unroll
        for (int n = 0; n < P1; ++n) x[n] = mk(0.0, 0.0);
        if (id >= 0) {
#pragma unroll
            for (int n = 0; n < P1; ++n) x[n] = w[(int64_t)n * nbox];
        }
    }
#pragma unroll 1
    for (int k = 0; k < nlev; ++k) {
        if (!zero) {
            const int q = (lane >> (2 * k)) & 3;
            const double ex = (q & 1) ? 0.5 : -0.5, ey = (q & 2) ? 0.5 : -0.5;
            band_rotate<P1>(x, -ex, ey);  // (2 u)^-m with u = -eps
            band_toeplitz_up<P1>(x);
            band_rotate<P1>(x, -ex, -ey);  // u^n
            band_sum<P1>(x, k);
        }
        id = tab[(k + 1) * 64];
        const int b = id & (kBandNonLeaf - 1);
        if (id >= 0 && !(id & kBandNonLeaf)) {  // a leaf brings its own multipole
            const cplx *w = W + b;
#pragma unroll
            for (int n = 0; n < P1; ++n) x[n] = w[(int64_t)n * nbox];
        } else if (id >= 0) {
            // the lanes of the box share its stores
            const int G = 4 << (2 * k), s = lane & (G - 1);
            cplx *w = W + b;
#pragma unroll
            for (int n = 0; n < P1; ++n)
                if ((n & (G - 1)) == s) w[(int64_t)n * nbox] = x[n];
        }
        zero = __ballot(id >= 0) == 0;
    }
}

// loc: local of the pass (vector and, with a complex impedance, H or G) from blockIdx.y
template <int PB>
__global__ __launch_bounds__(256) void k_l2l_band(int nwave, int nlev, const int32_t *__restrict__ tab, int nbox,
                                                  cplx *__restrict__ Lam) {
    constexpr int P1 = PB + 1;
    const int wv = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (wv >= nwave) return;
    const int lane = threadIdx.x & 63;
    Lam += (int64_t)blockIdx.y * P1 * nbox;
    tab += (int64_t)wv * (nlev + 1) * 64 + lane;
    cplx x[P1];
    {
        const int id = tab[nlev * 64];
        const cplx *l = Lam + (id >= 0 ? id & (kBandNonLeaf - 1) : 0);
#pragma unroll
        for (int n = 0; n < P1; ++n) x[n] = mk(0.0, 0.0);
        if (id >= 0) {
#pragma unroll
            for (int n = 0; n < P1; ++n) x[n] = l[(int64_t)n * nbox];
        }
    }
#pragma unroll 1
    for (int k = nlev - 1; k >= 0; --k) {
        const int id = tab[k * 64];
        if (__ballot(id >= 0) == 0) break;  // nothing below either
        const int q = (lane >> (2 * k)) & 3;
        const double ex = (q & 1) ? 0.5 : -0.5, ey = (q & 2) ? 0.5 : -0.5;
        band_rotate<P1>(x, ex, ey);  // eps^n
        band_toeplitz_down<P1>(x);
        band_rotate<P1>(x, ex, -ey);  // (2 eps)^-m
        if (id >= 0) {
            const int G = 1 << (2 * k), s = lane & (G - 1);
            cplx *l = Lam + (id & (kBandNonLeaf - 1));
            // every lane of the box adds its own local; they share the stores once all have read it
#pragma unroll
            for (int n = 0; n < P1; ++n) x[n] += l[(int64_t)n * nbox];
#pragma unroll
            for (int n = 0; n < P1; ++n)
                if ((n & (G - 1)) == s) l[(int64_t)n * nbox] = x[n];
        }
    }
}

}  // namespace fmmhp
