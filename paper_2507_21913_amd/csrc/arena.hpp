// Device memory of a plan: the arena its arrays come from, and the growth of its workspaces.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>
#include <initializer_list>
#include <vector>

#include "../../include/fmmhp.h"

namespace fmmhp {

void set_error(const char *fmt, ...);

// Device allocations owned by one plan.  Arrays share slabs (a plan holds some 90 arrays; a hipMalloc and
// a hipFree for each took 5 of the 11 ms of a 200,000-point training step): a slab is twice as large as
// everything allocated so far, from 1 to 64 MB; an array that does not fit one has an allocation of its
// own.  Nothing is given back before the plan's end: a recorded graph may hold any of the addresses.
struct Arena {
    std::vector<void *> ptrs;  // slabs and large arrays
    int64_t bytes = 0;         // requested
    int64_t held = 0;          // taken from the device
    int tries = 0;             // requests (FMMHP_TEST_FAIL_ALLOC counts them)
    char *cur = nullptr;       // the open slab
    size_t left = 0;

    struct Part {
        void **p;
        size_t bytes;
    };

    // Several arrays at once: all of them, or none and nothing taken (the pointers are left alone then).
    // Arrays that fit the open slab go there, the others share one new allocation.
    fmmhp_status alloc_all(std::initializer_list<Part> parts, const char *what) {
        size_t total = 0, placed = 0, rest = 0;  // placed: in the open slab
        for (const Part &a : parts) {
            const size_t need = padded(a.bytes);
            total += a.bytes;
            (placed + need <= left ? placed : rest) += need;
        }
        ++tries;
        if (const char *e = getenv("FMMHP_TEST_FAIL_ALLOC")) {  // "k": the k-th request fails; "k+": every one from it on
            char *end = nullptr;
            const long k = strtol(e, &end, 10);
            if (k > 0 && (tries == k || (*end == '+' && tries > k))) {
                set_error("allocation of %s (%zu bytes, array %d of the plan) failed (test hook)", what, total, tries);
                return FMMHP_ENOMEM;
            }
        }
        char *more = nullptr;
        size_t got = 0;
        if (rest > 0) {
            const size_t slab = std::min<size_t>((size_t)64 << 20, std::max<size_t>((size_t)1 << 20, 2 * ((size_t)bytes + placed)));
            got = std::max(rest, slab);
            hipError_t e = take(&more, got);
            if (e != hipSuccess && got > rest) e = take(&more, got = rest);  // no room for a slab: the arrays alone
            if (e != hipSuccess) {
                set_error("hipMalloc of %s (%zu bytes) failed: %s", what, total, hipGetErrorString(e));
                return FMMHP_ENOMEM;
            }
            ptrs.push_back(more);
            held += (int64_t)got;
        }
        char *m = more;
        for (const Part &a : parts) {
            const size_t need = padded(a.bytes);
            char *&at = need <= left ? cur : m;
            if (need <= left) left -= need;
            *a.p = at;
            at += need;
        }
        if (got - rest > left) {  // the new slab is the open one
            cur = m;
            left = got - rest;
        }
        bytes += (int64_t)total;
        return FMMHP_OK;
    }

    fmmhp_status alloc(void **p, size_t nbytes, const char *what) { return alloc_all({Part{p, nbytes}}, what); }
    template <class T>
    fmmhp_status alloc_n(T **p, size_t n, const char *what) {
        return alloc((void **)p, (n ? n : 1) * sizeof(T), what);
    }

    void release() {
        for (void *p : ptrs) (void)hipFree(p);
        *this = Arena();
    }

private:
    static size_t padded(size_t nbytes) { return (nbytes + 255) / 256 * 256; }
    static hipError_t take(char **m, size_t nbytes) {
        const hipError_t e = hipMalloc((void **)m, nbytes);
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
    }
};

template <class T>
inline Arena::Part part(T **p, size_t n) {
    return Arena::Part{(void **)p, (n ? n : 1) * sizeof(T)};
}

// Grows a workspace of cap vectors to want, or to half, a quarter, ... of it where the memory is short:
// grow(w) makes it w wide, or returns FMMHP_ENOMEM and changes nothing.  A width that failed is not tried
// again (limit).  Fails only where not even one vector has a place.
template <class Grow>
inline fmmhp_status widen(int want, int cap, int &limit, Grow &&grow) {
    for (int w = std::min(want, limit); w > cap;) {
        const fmmhp_status st = grow(w);
        if (st != FMMHP_ENOMEM || w == 1) return st;
        limit = w /= 2;
    }
    return FMMHP_OK;
}

}  // namespace fmmhp
