// Pieces shared by the C-ABI translation units: the context, error reporting
// and graph recording.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <string>

#include <cmath>
#include <thread>

#include "graph.h"
#include "kernels.h"
#include "kfbi.h"

namespace kfbi {

// The message of the last error on this host thread (kfbi_last_error).
std::string& last_error();

inline kfbi_status set_err(kfbi_status s, const std::string& msg) {
    last_error() = msg;
    return s;
}

inline kfbi_status check_ptr(const void* p, const char* name) {
    if (!p) return set_err(KFBI_ERR_ARG, std::string(name) + " is NULL");
    return KFBI_OK;
}

// Constants of the tridiagonal solve along x of one sine mode (Alg. 4): after
// the transforms along the other axes, h^2 (L_h - kappa) acts on a row as
// v_{i-1} - (2 + d) v_i + v_{i+1}, with d = h^2 kappa + 4 sin^2 of each other
// axis' mode angle (> 0).
inline ModeConst row_solve_constants(double d, int N) {
    const int C = N / 64;
    const double sq = std::sqrt(d * (4.0 + d));
    const double r = 1.0 + 0.5 * d - 0.5 * sq;             // root of r^2 - (2 + d) r + 1 in (0, 1)
    ModeConst c{};
    c.r = r;
    c.rinv = 1.0 / r;
    c.logr = std::log1p(0.5 * d - 0.5 * sq);
    c.rC = std::pow(r, C);
    c.rH = std::pow(r, modes_chunk(N));
    c.rN1 = std::exp((N - 1.0) * c.logr);
    const double r2N = std::exp(2.0 * N * c.logr);
    c.smc = -r / (1.0 - r2N);
    return c;
}

// The host's end of a GMRES run's GmresPub: pinned, coherent host memory.
struct GmresHost {
    GmresPub* pub = nullptr;
    unsigned epoch = 0;                                      // of the run in flight

    kfbi_status alloc() {
        if (hipHostMalloc((void**)&pub, sizeof(GmresPub), hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
            hipGetLastError();
            pub = nullptr;
            return set_err(KFBI_ERR_OOM, "pinned host allocation of the GMRES state mirror failed");
        }
        *pub = GmresPub{};
        return KFBI_OK;
    }
    void free() {
        if (pub) hipHostFree(pub);
        pub = nullptr;
    }
    unsigned next_epoch() { return epoch = epoch + 1 ? epoch + 1 : 1; }
    bool over() const { return __atomic_load_n(&pub->done, __ATOMIC_ACQUIRE) == epoch; }
    unsigned again() const { return __atomic_load_n(&pub->again, __ATOMIC_RELAXED); }
    // slots of this run whose commit has run, of `launched`; *last: the next one is
    // expected to end it
    long long committed(long long launched, bool* last) const {
        const unsigned long long v = __atomic_load_n(&pub->prog, __ATOMIC_RELAXED);
        if ((unsigned)(v >> 32) != epoch) {
            *last = false;
            return 0;
        }
        *last = ((unsigned)v & kGmLastSlot) != 0;
        return launched - (((unsigned)launched - (unsigned)v) & (kGmLastSlot - 1));
    }
};

// A bound of a GMRES run's slots.  A step takes one and its second Gram-Schmidt pass
// another; a cycle takes two more, the one in which its end is found and the
// residual's, and a cycle can be one step long: its estimate passes the tolerance where
// the true residual, held up by rounding, does not.  Besides, the first residual.
inline long long gmres_slot_bound(int max_iter) { return 4LL * max_iter + 8; }

// Runs the slots of a run that may stop early: `enqueue` launches one slot on the
// stream.  A slot is launched while the one before it runs, as soon as the commit
// before that is known, and none beyond the one expected to end the run; so the
// device does not wait for the host between slots and no launched slot finds the run
// over.  (Replayed graphs of several slots, polled in between, launched up to half of
// their slots for nothing, 5 us each, and a poll left the device idle for 25 us; a
// slot launched by itself takes 1 us more than in a graph.)  `drive` does what can be
// done now; several runs may be driven in turn.
struct GmresDriver {
    GmresHost* host = nullptr;
    hipStream_t stream = nullptr;
    // 64 bits: a cap of 2^30 iterations ("no cap") is a bound of more slots than an int holds
    long long launched = 0, most = 0;                        // most: see gmres_slot_bound
    long long held = 0;                                      // the commit that announced the end (0: none)
    unsigned again = 0;                                      // residuals seen before that
    unsigned spins = 0;
    bool idle = false;                                       // the stream was seen empty after the last launch

    template <class F>
    kfbi_status drive(F enqueue, bool* over) {
        *over = host->over();
        if (*over) return KFBI_OK;
        bool last = false;
        const unsigned seen = host->again();                 // before the commit: a residual in between counts as new
        long long done = host->committed(launched, &last);
        if (idle) {                                          // everything launched has run
            done = launched;
            held = 0;
        } else if (last && held != done) {
            held = done;
            again = seen;
        }
        const bool hold = held && launched > held && host->again() == again;
        if (launched - done <= 1 && !hold) {
            if (launched >= most) {                          // never: the device ends every run before
                const hipError_t e = hipStreamSynchronize(stream);
                if (e != hipSuccess) return set_err(KFBI_ERR_DEVICE, hipGetErrorString(e));
                if ((*over = host->over())) return KFBI_OK;
                return set_err(KFBI_ERR_DEVICE, "a GMRES run did not end");
            }
            spins = 0;
            idle = false;
            launched += 1;
            return enqueue(stream);
        }
        // waiting: now and then ask the runtime, so that a failed stream is found
        // and none is waited for in vain
        if ((++spins & 0x3ff) == 0) {
            const hipError_t e = hipStreamQuery(stream);
            if (e == hipErrorNotReady) {
                hipGetLastError();
            } else if (e != hipSuccess) {
                return set_err(KFBI_ERR_DEVICE, hipGetErrorString(e));
            } else {
                idle = true;
            }
        }
        std::this_thread::yield();
        return KFBI_OK;
    }
};

// Record what `enqueue(stream)` launches as the nodes of a new graph (see
// graph.h: no stream capture) and instantiate it.  Returns false (and leaves
// *out null) if recording or instantiation fails; the caller then launches
// directly.  `enqueue` must issue kernel launches only.
template <class F>
bool record_graph(hipStream_t stream, hipGraphExec_t* out, F enqueue) {
    *out = nullptr;
    GraphRec rec;
    if (hipGraphCreate(&rec.graph, 0) != hipSuccess) {
        hipGetLastError();
        return false;
    }
    graph_rec() = &rec;
    const kfbi_status e = enqueue(stream);
    graph_rec() = nullptr;
    const bool ok = e == KFBI_OK && rec.last != nullptr &&
                    hipGraphInstantiate(out, rec.graph, nullptr, nullptr, 0) == hipSuccess;
    if (!ok) {
        hipGetLastError();
        *out = nullptr;
    }
    hipGraphDestroy(rec.graph);
    return ok;
}

}  // namespace kfbi

#define HIP_TRY(expr)                                                                                   \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess)                                                                           \
            return ::kfbi::set_err(KFBI_ERR_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

namespace kfbi {

// Arguments of one Neumann solve (device pointers, as kfbi_solve_neumann).
struct NeumannIO {
    const double *f_grid, *f_gamma, *g_n;
    double *u_grid, *u_gamma, *dn_gamma, *psi;
};

// Two Neumann solves whose problems enqueue on different streams, overlapped:
// the volume potentials, then GMRES batches on both with the host reading both
// states after each round, then the final solves.  Leaves the final solves
// enqueued (no wait at the end).  KFBI_NOT_CONVERGED if either hit its cap.
kfbi_status solve_neumann_pair(kfbi_prob* pa, const NeumannIO& ia, kfbi_prob* pb, const NeumannIO& ib, int* iters_a,
                               int* iters_b);

}  // namespace kfbi

struct kfbi_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    size_t lds_max = 65536;
    int num_cu = 256;
    std::atomic<int> users{1};          // its creator, and every object made in it
};

namespace kfbi {

inline void ctx_release(kfbi_ctx* c) {
    if (!c || --c->users) return;
    if (c->own_stream) hipStreamDestroy(c->stream);
    delete c;
}

// An object's hold on its context: a caller (a garbage collector that finalises a
// cycle in any order) may destroy the context first.
class CtxRef {
public:
    CtxRef() = default;
    CtxRef(const CtxRef&) = delete;
    CtxRef& operator=(const CtxRef&) = delete;
    ~CtxRef() { ctx_release(c_); }
    void operator=(kfbi_ctx* c) {
        if (c) ++c->users;
        ctx_release(c_);
        c_ = c;
    }
    kfbi_ctx* operator->() const { return c_; }
    operator kfbi_ctx*() const { return c_; }

private:
    kfbi_ctx* c_ = nullptr;
};

}  // namespace kfbi
