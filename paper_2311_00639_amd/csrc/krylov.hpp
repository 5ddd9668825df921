// Lanczos propagator and the small tridiagonal exponential (host side).
#pragma once

#include <complex>
#include <vector>

#include "internal.hpp"

namespace syk {

bool tridiag_eig(int n, std::vector<double> &d, std::vector<double> e, std::vector<double> &Z);

// a-posteriori error of a Lanczos run: |[e^{z T} e_1]_n| from the eigenvalues of T and the first
// and last components of its eigenvectors only (O(n^2) instead of the O(n^3) of TriExp)
class TriLast {
  public:
    TriLast(int n, const double *alpha, const double *beta_off);
    bool ok() const { return ok_; }
    double last(std::complex<double> z) const;

  private:
    bool ok_ = false;
    std::vector<double> lam_, w_;        // eigenvalues, products of first and last components
};

// e^{z T} e_1 for a real symmetric tridiagonal T, through T = Z diag(lam) Z^T
class TriExp {
  public:
    TriExp(int n, const double *alpha, const double *beta_off);
    bool ok() const { return ok_; }
    void apply(std::complex<double> z, std::complex<double> *c) const;   // all n components
    std::complex<double> last(std::complex<double> z) const;             // component n-1

  private:
    int n_;
    bool ok_ = false;
    std::vector<double> lam_, Z_;
};

// Argument checks of Krylov options (throws SYK_EINVAL).
void check_krylov_opts(const syk_krylov_opts &o);

size_t krylov_workspace_bytes(uint64_t n, int m, size_t elem_bytes);

// Optional timing of apply_H launches with HIP events recorded on the launch stream.
// Pairs are read back (flush) only after the stream has been synchronised.
class ApplyTimer {
  public:
    ~ApplyTimer();
    void begin(hipStream_t s);
    void end(hipStream_t s);
    void flush();              // the stream must be synchronised
    double ms = 0.0;
    long long launches = 0;

  private:
    std::vector<hipEvent_t> pool_;
    size_t used_ = 0;
};

// Scalars that kernels store to pinned host memory and the host polls for, so that it can follow a
// Lanczos run without waiting for the stream: coherent memory, written with system-scope atomic
// stores, one 8-byte value per slot, so that no order between slots is needed.  Blocks come from a pool shared by all threads (one
// per run in progress), which syk_release_workspace empties.
class HostScalars {
  public:
    static constexpr int kSlots = 2 * 132;      // one Lanczos run: alpha_j, then ||u_j||^2
    HostScalars();
    ~HostScalars();                             // the stream must not hold work that stores here
    HostScalars(const HostScalars &) = delete;
    HostScalars &operator=(const HostScalars &) = delete;
    // slots of the next Lanczos run, marked empty.  Two sets alternate: kernels of the run before
    // may still store to the other set, those of the run before that are done (the run in
    // between read a value that a later kernel of the stream stored).
    void next();
    double *alpha(int j) const { return p_ + set_ * kSlots + j; }
    double *norm2(int j) const { return p_ + set_ * kSlots + kSlots / 2 + j; }
    double *dev(double *host) const { return dev_ + (host - p_); }
    // the value of a slot, waiting until a kernel on `s` has stored it
    double wait(const double *slot, hipStream_t s) const;
    static void trim();                         // free the idle blocks

  private:
    double *p_ = nullptr, *dev_ = nullptr;
    int set_ = 0;
};

template <typename T>
class KrylovRun {
  public:
    // ws: device workspace of at least krylov_workspace_bytes(n, m, sizeof(T)) bytes
    // rot: layout rotation of the vectors (0 = standard index order)
    KrylovRun(Hamiltonian &h, int blk, int rot, uint64_t n, int m, char *ws, hipStream_t s);
    ~KrylovRun();                               // waits for the stream where work may be left on it
    // out = e^{z H} v (out may be v, or overlap it); accumulates into st.  The result is enqueued, not waited for.
    void run(std::complex<double> z, const T *v, T *out, const syk_krylov_opts &o, syk_krylov_stats &st);
    double norm(const T *v);
    void set_timer(ApplyTimer *t) { timer_ = t; }
    double *partials() { return partials_; }
    double *scratch() { return scratch_; }
    int n_part() const { return n_part_; }

  private:
    T *vec(int j) { return basis_ + static_cast<size_t>(j) * vec_stride_ * 2; }
    void copy(const T *v, T *out);
    // reorth = 0: fused steps, the host a step or two ahead of the last one it has checked
    int next_check(int k) const;
    LanczosStep<T> step_of(int j, const T *u0);
    void enqueue_one(int j, const T *u0);
    void close(int j, const T *u0);
    void run_fused(std::complex<double> z, const T *v, T *out, const syk_krylov_opts &o, syk_krylov_stats &st);
    void run_plain(std::complex<double> z, const T *v, T *out, const syk_krylov_opts &o, syk_krylov_stats &st);
    // enqueue fused Lanczos step j from u_j (slot 0: u0)
    void enqueue(int j, const T *u0);
    // largest fraction f <= remaining of the sub-step with err(f) <= tol f
    template <typename E>
    static double bisect(const E &err, double remaining, double tol);
    // one unfused Lanczos step; returns true if w was fully reorthogonalised
    bool iterate(int j, int reorth);
    // reorth = 3: update the estimates of |<v_{j+1}, v_k>| from alpha, beta; true if a
    // full reorthogonalisation is due
    bool partial_estimate(int j);

    Hamiltonian &h_;
    int blk_, rot_;
    uint64_t n_;
    int m_;
    hipStream_t s_;
    size_t vec_stride_ = 0;    // complex elements between basis vectors
    T *basis_ = nullptr;
    double *partials_ = nullptr, *alpha_ = nullptr, *beta2_ = nullptr, *coef_ = nullptr, *scratch_ = nullptr;
    double *fused_ = nullptr, *norms_ = nullptr;
    bool tiled_ = false;                  // the tiled kernel serves the block
    bool plain_ = false;                  // H is too small or large for unnormalised vectors
    bool one_ = false;                    // one launch per step
    int n_step_ = 0;                      // its workgroups
    bool big_ = false;                    // tiled, more than 2^21 amplitudes
    int n_norm_ = 0;                      // partials of ||u||^2
    HostScalars host_;
    bool pending_ = false;                // the stream may hold steps that store to host_
    // partial reorthogonalisation state: omega_[0] row j - 1, omega_[1] row j of the
    // estimated <v_j, v_k>; host copies of alpha and beta; whether the next step must be
    // reorthogonalised too
    std::vector<double> omega_[2], ha_, hb_;
    double anorm_ = 0.0;
    bool force_next_ = false;
    int n_part_ = 0;
    ApplyTimer *timer_ = nullptr;
};

}  // namespace syk
