// Workspaces that a plan's evaluations grow on demand, each as a whole: where that fails, the workspace
// stays what it was, and what fitted before still runs.
#pragma once
#include "internal.hpp"

namespace fmmhp {

// Row length of a source in the FP32 M2L: 2(p+1) embedded coefficients, the low parts of Re w_0 and
// Im w_0, zero padding to a multiple of 4.
__host__ __device__ constexpr int m2l32_kp(int PB) { return ((2 * (PB + 1) + 2 + 3) / 4) * 4; }

constexpr int kWsArrays = 8;

// Bytes of the arrays of a pass workspace for nv vectors (W, Lam, qs, near, red, rank1, Wf, part; 0: not in
// use).
inline void vec_ws_sizes(const Tree &T, const Sched &S, int nv, size_t (&b)[kWsArrays]) {
    const size_t nb = (size_t)T.nbox, P1 = (size_t)S.PB + 1;
    b[0] = nv * P1 * nb * sizeof(cplx);
    b[1] = nv * (size_t)S.nloc * P1 * nb * sizeof(cplx);
    b[2] = nv * (size_t)T.n * sizeof(double);
    b[3] = nv * (size_t)T.n * sizeof(double2);
    b[4] = nv * (size_t)S.n_rch * sizeof(cplx);
    b[5] = nv * (size_t)T.n_inst * sizeof(cplx);
    b[6] = S.m2l_fp32 ? nv * nb * (size_t)m2l32_kp(S.PB) * sizeof(float) : 0;
    b[7] = S.sym_ok && (S.near_walk == 3 || S.near_walk == 4) ? nv * (size_t)S.sym_npart * sizeof(double) : 0;
}

// Bytes of a pass workspace for nv vectors (each array aligned to 256 bytes); carves it from base
// when base is given.
inline size_t vec_ws_layout(const Tree &T, const Sched &S, int nv, unsigned char *base, VecWs *w) {
    size_t sizes[kWsArrays], off[kWsArrays], at = 0;
    vec_ws_sizes(T, S, nv, sizes);
    for (int k = 0; k < kWsArrays; ++k) {
        off[k] = at;
        at += (sizes[k] + 255) / 256 * 256;
    }
    if (base) {
        w->cap = nv;
        w->W = (cplx *)(base + off[0]);
        w->Lam = (cplx *)(base + off[1]);
        w->qs = (double *)(base + off[2]);
        w->near = (double2 *)(base + off[3]);
        w->red = (cplx *)(base + off[4]);
        w->rank1 = (cplx *)(base + off[5]);
        w->Wf = sizes[6] ? (float *)(base + off[6]) : nullptr;
        w->part = sizes[7] ? (double *)(base + off[7]) : nullptr;
    }
    return at;
}

// Per-vector workspace (multipoles, locals, sorted charges, near-field sums, surface sums) for nv
// vectors at once; grown on demand, owned by the plan.  Where one array has no place, the workspace
// stays what it was.
inline fmmhp_status ensure_vec_ws(Arena &A, const Tree &T, Sched &S, int nv) {
    if (S.ws.cap >= nv) return FMMHP_OK;
    size_t b[kWsArrays];
    vec_ws_sizes(T, S, nv, b);
    VecWs w;
    FMMHP_CHECK(A.alloc_all({Arena::Part{(void **)&w.W, b[0]}, Arena::Part{(void **)&w.Lam, b[1]},
                             Arena::Part{(void **)&w.qs, b[2]}, Arena::Part{(void **)&w.near, b[3]},
                             Arena::Part{(void **)&w.red, b[4]}, Arena::Part{(void **)&w.rank1, b[5]},
                             Arena::Part{(void **)&w.Wf, b[6]}, Arena::Part{(void **)&w.part, b[7]}},
                            "pass workspace"));
    if (!b[6]) w.Wf = nullptr;
    if (!b[7]) w.part = nullptr;
    w.cap = nv;
    S.ws = w;
    return FMMHP_OK;
}

// Partial sums of the symmetric near-field walk for the plan's workspace, allocated when the walk is
// in use (walk 3 or 4 on a plan whose lists allow it).
inline fmmhp_status ensure_sym_part(Arena &A, Sched &S) {
    if (!((S.near_walk == 3 || S.near_walk == 4) && S.sym_ok) || S.ws.part) return FMMHP_OK;
    return A.alloc_n(&S.ws.part, (size_t)S.ws.cap * S.sym_npart, "near-field pair partial sums");
}

// Widest pass that nvec vectors take.
inline int pass_width(int nvec) { return nvec >= 8 ? 8 : nvec >= 4 ? 4 : nvec >= 2 ? 2 : 1; }

// Workspace for the widest passes that nvec vectors take; where the memory is short, for narrower ones.
inline fmmhp_status ensure_eval_ws(Arena &A, const Tree &T, Sched &S, int nvec) {
    return widen(pass_width(nvec), S.ws.cap, S.ws_limit, [&](int w) { return ensure_vec_ws(A, T, S, w); });
}

// Whether s records a graph.  A workspace is then taken as it is: an allocation is refused there.
inline bool recording(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

// Lets this thread allocate while another stream or thread records a graph.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    RelaxedCapture(const RelaxedCapture &) = delete;
    RelaxedCapture &operator=(const RelaxedCapture &) = delete;
};

// ensure_eval_ws for a call on s: narrower passes rather than an allocation within a recording.
inline fmmhp_status grow_eval_ws(Arena &A, const Tree &T, Sched &S, int nvec, hipStream_t s) {
    if (S.ws.cap >= std::min(pass_width(nvec), S.ws_limit) || recording(s)) return FMMHP_OK;
    RelaxedCapture relaxed;
    return ensure_eval_ws(A, T, S, nvec);
}

// Split charges and the potentials of their parts, for g complex vectors.
inline fmmhp_status ensure_split(Arena &A, const Tree &T, Sched &S, int g) {
    if (S.ccap >= g) return FMMHP_OK;
    FMMHP_CHECK(A.alloc_all({part(&S.cq, (size_t)2 * g * T.n), part(&S.cphi, (size_t)4 * g * T.n)},
                            "complex-charge workspace"));
    S.ccap = g;
    return FMMHP_OK;
}

// Split workspace of a call of nvec complex vectors on s: up to four at once (one pass of eight real ones);
// where the memory is short, fewer, and within a recording those that there are.
inline fmmhp_status grow_split(Arena &A, const Tree &T, Sched &S, int nvec, hipStream_t s) {
    auto grow = [&](int g) { return ensure_split(A, T, S, g); };
    if (S.ccap >= std::min(nvec, S.ccap_limit)) return FMMHP_OK;
    if (recording(s)) return grow(1);  // (a refusal there says nothing about the memory)
    RelaxedCapture relaxed;
    return widen(std::min(nvec, kVecChunk / 2), S.ccap, S.ccap_limit, grow);
}

inline fmmhp_status ensure_bwd(Arena &A, const Tree &T, Sched &S) {
    if (S.bw.ready) return FMMHP_OK;
    const size_t n = (size_t)T.n;
    BwdWork &b = S.bw;
    FMMHP_CHECK(A.alloc_all({part(&b.q3, 3 * n), part(&b.qc, n), part(&b.phi3, 3 * n), part(&b.gx3, 3 * n),
                             part(&b.gy3, 3 * n), part(&b.near_gx, 3 * n), part(&b.near_gy, 3 * n),
                             part(&b.red, (size_t)S.n_rch + T.n_inst)},
                            "adjoint workspace"));
    b.ready = true;
    return FMMHP_OK;
}

}  // namespace fmmhp
