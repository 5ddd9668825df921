// Lanczos propagator out = e^{z H_blk} v (the restarted Krylov time evolution of
// supplement Sec. I.A), with a-posteriori step control.
//
// One sub-step: Lanczos on the normalised start vector builds V_k and the real symmetric
// tridiagonal T_k (alpha_j = Re <v_j, H v_j - beta_{j-1} v_{j-1}>, beta_j = ||w_j||, both
// reduced in double on the device).  The small exponential c(tau) = e^{tau z T_k} e_1 comes
// from the eigendecomposition of T_k (implicit QL, double).  The estimate
// err(tau) = beta_k |c_{k-1}(tau)| bounds the error of ||v|| V_k c(tau) relative to ||v||
// (Saad 1992).  A sub-step of fraction tau of z is accepted when err(tau) <= tol * tau,
// so accepted errors sum to at most tol.  beta_k ~ 0 means V_k spans an invariant
// subspace and the result is exact.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <complex>
#include <cstring>
#include <mutex>
#include <thread>

#include "krylov.hpp"

namespace syk {

// ------------------------------------------------------------------ tridiagonal eigensolver
// Implicit QL iteration with shifts for a real symmetric tridiagonal matrix (Bowdler,
// Martin, Reinsch & Wilkinson, Numer. Math. 11 (1968)): d <- eigenvalues, Z <- orthonormal
// eigenvectors (column k of Z, row-major).  e[i] couples d[i] and d[i+1].  Z holds `rows` rows of
// the identity on entry (all n of them, or those whose eigenvector components are wanted).
static bool tridiag_ql(int n, std::vector<double> &d, std::vector<double> e, std::vector<double> &Z, int rows) {
    e.resize(n, 0.0);
    e[n - 1] = 0.0;
    const double eps = 2.220446049250313e-16;
    for (int l = 0; l < n; ++l) {
        int iter = 0;
        for (;;) {
            int m = l;
            for (; m < n - 1; ++m) {
                const double dd = std::fabs(d[m]) + std::fabs(d[m + 1]);
                if (std::fabs(e[m]) <= eps * dd) break;
            }
            if (m == l) break;
            if (++iter > 200) return false;
            // shift: eigenvalue of the leading 2x2 block closest to d[l]
            double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
            double r = std::hypot(g, 1.0);
            g = d[m] - d[l] + e[l] / (g + std::copysign(r, g));
            double s = 1.0, c = 1.0, p = 0.0;
            int i = m - 1;
            bool deflated = false;
            for (; i >= l; --i) {
                const double f = s * e[i];
                const double b = c * e[i];
                r = std::hypot(f, g);
                e[i + 1] = r;
                if (r == 0.0) {          // underflow: split here and restart the sweep
                    d[i + 1] -= p;
                    e[m] = 0.0;
                    deflated = true;
                    break;
                }
                s = f / r;
                c = g / r;
                g = d[i + 1] - p;
                r = (d[i] - g) * s + 2.0 * c * b;
                p = s * r;
                d[i + 1] = g + p;
                g = c * r - b;
                for (int k = 0; k < rows; ++k) {
                    double *row = &Z[static_cast<size_t>(k) * n];
                    const double zf = row[i + 1];
                    row[i + 1] = s * row[i] + c * zf;
                    row[i] = c * row[i] - s * zf;
                }
            }
            if (deflated) continue;
            d[l] -= p;
            e[l] = g;
            e[m] = 0.0;
        }
    }
    return true;
}

bool tridiag_eig(int n, std::vector<double> &d, std::vector<double> e, std::vector<double> &Z) {
    Z.assign(static_cast<size_t>(n) * n, 0.0);
    for (int i = 0; i < n; ++i) Z[static_cast<size_t>(i) * n + i] = 1.0;
    return tridiag_ql(n, d, std::move(e), Z, n);
}

TriLast::TriLast(int n, const double *alpha, const double *beta_off) : lam_(alpha, alpha + n), w_(n) {
    std::vector<double> e(std::max(n, 1), 0.0), Z(2 * static_cast<size_t>(n), 0.0);
    for (int i = 0; i + 1 < n; ++i) e[i] = beta_off[i];
    Z[0] = 1.0;                                    // row 0 and row n - 1 of the identity
    Z[2 * static_cast<size_t>(n) - 1] = 1.0;
    ok_ = tridiag_ql(n, lam_, std::move(e), Z, 2);
    for (int k = 0; k < n; ++k) {
        w_[k] = Z[k] * Z[static_cast<size_t>(n) + k];
        if (!std::isfinite(lam_[k])) ok_ = false;
    }
}

double TriLast::last(std::complex<double> z) const {
    std::complex<double> acc = 0.0;
    for (size_t k = 0; k < lam_.size(); ++k) acc += std::exp(z * lam_[k]) * w_[k];
    return std::abs(acc);
}

TriExp::TriExp(int n, const double *alpha, const double *beta_off) : n_(n) {
    lam_.assign(alpha, alpha + n);
    std::vector<double> e(std::max(n, 1), 0.0);
    for (int i = 0; i + 1 < n; ++i) e[i] = beta_off[i];
    ok_ = tridiag_eig(n, lam_, e, Z_);
    for (double v : lam_)
        if (!std::isfinite(v)) ok_ = false;
}

// c = Z diag(e^{z lam}) Z^T e_1
void TriExp::apply(std::complex<double> z, std::complex<double> *c) const {
    std::vector<std::complex<double>> w(n_);
    for (int k = 0; k < n_; ++k) w[k] = std::exp(z * lam_[k]) * Z_[k];          // Z[0][k] = Z_[k]
    for (int i = 0; i < n_; ++i) {
        std::complex<double> acc = 0.0;
        const double *row = &Z_[static_cast<size_t>(i) * n_];
        for (int k = 0; k < n_; ++k) acc += row[k] * w[k];
        c[i] = acc;
    }
}

std::complex<double> TriExp::last(std::complex<double> z) const {
    std::complex<double> acc = 0.0;
    const double *row = &Z_[static_cast<size_t>(n_ - 1) * n_];
    for (int k = 0; k < n_; ++k) acc += row[k] * std::exp(z * lam_[k]) * Z_[k];
    return acc;
}

// ------------------------------------------------------------------ apply_H timing
ApplyTimer::~ApplyTimer() {
    for (auto e : pool_) ignore_status(hipEventDestroy(e));
}

void ApplyTimer::begin(hipStream_t s) {
    while (pool_.size() < used_ + 2) {
        hipEvent_t e;
        SYK_HIP(hipEventCreate(&e));
        pool_.push_back(e);
    }
    SYK_HIP(hipEventRecord(pool_[used_], s));
}

void ApplyTimer::end(hipStream_t s) {
    SYK_HIP(hipEventRecord(pool_[used_ + 1], s));
    used_ += 2;
}

void ApplyTimer::flush() {
    for (size_t k = 0; k + 1 < used_; k += 2) {
        float t = 0.0f;
        SYK_HIP(hipEventElapsedTime(&t, pool_[k], pool_[k + 1]));
        ms += t;
        launches += 1;
    }
    used_ = 0;
}

// ------------------------------------------------------------------ Lanczos driver
static int log2_of(uint64_t n) { return 63 - __builtin_clzll(n); }

void check_krylov_opts(const syk_krylov_opts &o) {
    auto require = [](bool c, const char *msg) {
        if (!c) fail(SYK_EINVAL, msg);
    };
    require(o.m >= 2 && o.m <= 128, "Krylov m must lie in [2, 128]");
    require(o.tol > 0.0 && std::isfinite(o.tol), "Krylov tol must be positive");
    require(o.reorth >= 0 && o.reorth <= 3, "reorth must be 0, 1, 2 or 3");
    require(o.max_substeps >= 0, "max_substeps must be >= 0");
}

// bytes from one Krylov basis vector to the next: the vector rounded up to 256 bytes plus
// 4 KiB, so that vectors read side by side (the recombination reads up to m of them at the
// same index) do not all start at the same low address bits (measured on a 60-vector
// recombination of 2^27 complex64 amplitudes: 11.7 ms against 12.9 ms with a stride of
// exactly 1 GiB)
static size_t basis_stride_bytes(uint64_t n, size_t elem_bytes) {
    return ((static_cast<size_t>(n) * 2 * elem_bytes + 255) & ~static_cast<size_t>(255)) + 4096;
}

// partial sums of the fused step: the apply's, one per workgroup, and, above 2^21 amplitudes in
// the same buffer once alpha_j is formed, the residual pass's, one per 256 amplitudes
constexpr uint64_t kBigBlock = 1ULL << 21;
static size_t fused_partials(uint64_t n) {
    return std::max<uint64_t>(lanczos_partials_max(log2_of(n)), n > kBigBlock ? n / 256 : 0);
}
// workgroups (and partial sums) of a residual pass up to 2^21 amplitudes, at most: every workgroup
// of the next pass may add them up
constexpr int kNormParts = 1024;
// workgroups of a one-launch step at most: two sets of three sums each fit the partials' space
constexpr int kStepGroups = 256;

size_t krylov_workspace_bytes(uint64_t n, int m, size_t elem_bytes) {
    const size_t vec = basis_stride_bytes(n, elem_bytes);
    const size_t part = static_cast<size_t>(reduction_blocks(n)) * 2 * (m + 2) * sizeof(double);
    const size_t scal = static_cast<size_t>(8 * (m + 4)) * sizeof(double);
    const size_t fused = (fused_partials(n) + kNormParts) * sizeof(double);
    auto up = [](size_t b) { return (b + 255) & ~static_cast<size_t>(255); };
    return static_cast<size_t>(m + 1) * up(vec) + up(part) + up(scal) + up(fused);
}

// The fused steps read v and the later basis vectors unnormalised, so that H u_j is formed at about c_max
// times the norm of u_j, which is ||v|| for j = 0 and of the order of c_max else (sums over u_j and H u_j
// at its third power).  Within these bounds on ||v|| and c_max nothing of that leaves the range
// of T (2^18 terms of 2^20 on a vector of 2^80 stay below 2^118), nor the sums that of a double.  The vectors
// grow in imaginary time: 2^80 leaves room for the chains of a correlator up to about beta = 45 at N = 56.
template <typename T>
static bool fused_norm(double s) {
    return sizeof(T) == 4 ? s >= 0x1p-40 && s <= 0x1p80 : s >= 0x1p-300 && s <= 0x1p300;
}
template <typename T>
static bool fused_terms(double c_max) {
    return sizeof(T) == 4 ? c_max >= 0x1p-40 && c_max <= 0x1p20 : c_max >= 0x1p-300 && c_max <= 0x1p300;
}

template <typename T>
KrylovRun<T>::KrylovRun(Hamiltonian &h, int blk, int rot, uint64_t n, int m, char *ws, hipStream_t s)
    : h_(h), blk_(blk), rot_(rot), n_(n), m_(m), s_(s) {
    auto up = [](size_t b) { return (b + 255) & ~static_cast<size_t>(255); };
    vec_stride_ = basis_stride_bytes(n, sizeof(T)) / (2 * sizeof(T));
    basis_ = reinterpret_cast<T *>(ws);
    char *p = ws + static_cast<size_t>(m + 1) * vec_stride_ * 2 * sizeof(T);
    n_part_ = reduction_blocks(n);
    partials_ = reinterpret_cast<double *>(p);
    p += up(static_cast<size_t>(n_part_) * 2 * (m + 2) * sizeof(double));
    alpha_ = reinterpret_cast<double *>(p);   // 2 (m+1)
    beta2_ = alpha_ + 2 * (m + 2);            // m+2
    coef_ = beta2_ + (m + 2);                 // 2 (m+2)
    scratch_ = coef_ + 2 * (m + 2);           // 2 (m+2)
    p += up(static_cast<size_t>(8 * (m + 4)) * sizeof(double));
    fused_ = reinterpret_cast<double *>(p);
    norms_ = fused_ + fused_partials(n);
    tiled_ = served_tiled<T>(h_, rot);
    big_ = n > kBigBlock && tiled_;
    plain_ = !tiled_ && !fused_terms<T>(h_.c_max);
    one_ = one_launch_steps<T>(h_);
    n_norm_ = static_cast<int>(std::min<uint64_t>(std::max<uint64_t>(n / 256, 1), big_ ? n / 256 : kNormParts));
}

template <typename T>
KrylovRun<T>::~KrylovRun() {
    // steps enqueued ahead of the last check may still store to the pinned scalars
    if (pending_) ignore_status(hipStreamSynchronize(s_));
}

// ------------------------------------------------------------------ pinned scalars
namespace {
std::mutex pin_mu;
std::vector<double *> *pin_pool() {
    static auto *v = new std::vector<double *>();   // never destroyed: no HIP calls at exit
    return v;
}
// what an empty slot holds: a NaN whose payload no arithmetic produces
const uint64_t kEmptySlot = 0x7ff8a5a5deadbeefULL;
}  // namespace

HostScalars::HostScalars() {
    {
        std::lock_guard<std::mutex> g(pin_mu);
        if (!pin_pool()->empty()) {
            p_ = pin_pool()->back();
            pin_pool()->pop_back();
        }
    }
    // coherent: a running kernel's store has to reach a polling host (any other flag alone leaves that
    // to the environment, HIP_HOST_COHERENT)
    if (!p_)
        SYK_HIP(hipHostMalloc(reinterpret_cast<void **>(&p_), 2 * kSlots * sizeof(double),
                              hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent));
    void *d = nullptr;
    const hipError_t e = hipHostGetDevicePointer(&d, p_, 0);
    if (e != hipSuccess) {
        std::lock_guard<std::mutex> g(pin_mu);
        pin_pool()->push_back(p_);
        hip_check(e, "hipHostGetDevicePointer");
    }
    dev_ = static_cast<double *>(d);
}

HostScalars::~HostScalars() {
    std::lock_guard<std::mutex> g(pin_mu);
    pin_pool()->push_back(p_);
}

void HostScalars::trim() {
    std::lock_guard<std::mutex> g(pin_mu);
    for (double *p : *pin_pool()) ignore_status(hipHostFree(p));
    pin_pool()->clear();
}

void HostScalars::next() {
    set_ ^= 1;
    for (int i = 0; i < kSlots; ++i) std::memcpy(p_ + set_ * kSlots + i, &kEmptySlot, sizeof(double));
}

double HostScalars::wait(const double *slot, hipStream_t s) const {
    const volatile uint64_t *q = reinterpret_cast<const volatile uint64_t *>(slot);
    uint64_t b;
    for (uint64_t spin = 0; (b = *q) == kEmptySlot; ++spin) {
        if (spin < 4096) {
            __builtin_ia32_pause();
            continue;
        }
        if (spin % 256 == 0) {
            // the kernel that stores the slot is on the stream: once the stream has drained
            // (or failed) there is nothing to wait for
            const hipError_t e = hipStreamQuery(s);
            if (e != hipErrorNotReady) {
                hip_check(e, "Lanczos step");
                b = *q;
                break;
            }
        }
        std::this_thread::yield();
    }
    double v;
    std::memcpy(&v, &b, sizeof v);
    return v;
}

template <typename T>
double KrylovRun<T>::norm(const T *v) {
    launch_norm2_partials<T>(v, n_, partials_, n_part_, s_);
    launch_reduce_partials(partials_, n_part_, 1, scratch_, s_);
    double h = 0.0;
    SYK_HIP(hipMemcpyAsync(&h, scratch_, sizeof(double), hipMemcpyDeviceToHost, s_));
    SYK_HIP(hipStreamSynchronize(s_));
    if (timer_) timer_->flush();
    if (!std::isfinite(h)) fail(SYK_ENUMERIC, "non-finite norm in Krylov propagation");
    return std::sqrt(h);
}

// one unfused Lanczos iteration j: fills slot j+1, alpha[j], beta2[j+1]
template <typename T>
bool KrylovRun<T>::iterate(int j, int reorth) {
    T *vj = vec(j);
    T *w = vec(j + 1);
    if (timer_) timer_->begin(s_);
    apply_block<T>(h_, blk_, rot_, vj, w, 1, n_, s_);
    if (timer_) timer_->end(s_);
    launch_lanczos_orth1<T>(w, j > 0 ? vec(j - 1) : nullptr, vj, beta2_ + j, n_, partials_, n_part_, s_);
    launch_reduce_partials(partials_, n_part_, 2, alpha_ + 2 * j, s_);
    launch_lanczos_orth2<T>(w, vj, alpha_ + 2 * j, n_, partials_, n_part_, s_);
    // reorth 1: one more pass against v_{j-1}, v_j; reorth 2: two full classical
    // Gram-Schmidt passes against v_0 .. v_j; reorth 3: the same two passes on the steps
    // where the estimated loss of orthogonality calls for them
    bool full = reorth == 2;
    if (reorth == 3) {
        launch_reduce_partials(partials_, n_part_, 1, beta2_ + j + 1, s_);
        full = partial_estimate(j);
    }
    if (reorth == 1 || full) {
        const int first = (reorth == 1) ? std::max(0, j - 1) : 0;
        const int nb = j + 1 - first;
        for (int pass = 0; pass < (full ? 2 : 1); ++pass) {
            launch_multi_dot_partials<T>(vec(first), vec_stride_, nb, w, n_, partials_, n_part_, s_);
            launch_reduce_partials(partials_, n_part_, 2 * nb, scratch_, s_);
            launch_subtract_proj<T>(w, vec(first), vec_stride_, nb, scratch_, n_, s_);
        }
        launch_norm2_partials<T>(w, n_, partials_, n_part_, s_);
    }
    launch_reduce_partials(partials_, n_part_, 1, beta2_ + j + 1, s_);
    launch_lanczos_normalize<T>(w, beta2_ + j + 1, n_, s_);
    return full;
}

// Partial reorthogonalisation (H. D. Simon, Math. Comp. 42 (1984) 115-142).  With
// normalised Lanczos vectors and beta_j v_{j+1} = H v_j - alpha_j v_j - beta_{j-1} v_{j-1},
// omega_{j,k} = <v_j, v_k> obeys
//   beta_j omega_{j+1,k} = beta_k omega_{j,k+1} + (alpha_k - alpha_j) omega_{j,k}
//                          + beta_{k-1} omega_{j,k-1} - beta_{j-1} omega_{j-1,k}
// up to rounding, which is modelled by adding 2 eps ||T|| with the sign of the sum
// (omega_{j,j} = 1, omega_{j+1,j} = eps).  When max_k |omega_{j+1,k}| exceeds sqrt(eps),
// v_{j+1} is reorthogonalised against every earlier vector, and so is v_{j+2} (the loss
// of v_{j+1} also reaches the next vector through the recurrence); the estimates of a
// reorthogonalised vector are reset to eps.  eps is the unit roundoff of the vectors.
template <typename T>
bool KrylovRun<T>::partial_estimate(int j) {
    const double eps = sizeof(T) == 4 ? 5.9604644775390625e-8 : 1.1102230246251565e-16;
    ha_.resize(static_cast<size_t>(m_) + 1);
    hb_.resize(static_cast<size_t>(m_) + 2);
    double ab[2];
    std::vector<double> b2(static_cast<size_t>(j) + 2);
    SYK_HIP(hipMemcpyAsync(ab, alpha_ + 2 * j, 2 * sizeof(double), hipMemcpyDeviceToHost, s_));
    SYK_HIP(hipMemcpyAsync(b2.data(), beta2_, (j + 2) * sizeof(double), hipMemcpyDeviceToHost, s_));
    SYK_HIP(hipStreamSynchronize(s_));
    ha_[j] = ab[0];
    for (int k = 0; k <= j; ++k) hb_[k] = std::sqrt(b2[k + 1]);   // beta_k = ||w_k||
    if (!std::isfinite(ha_[j]) || !std::isfinite(hb_[j])) fail(SYK_ENUMERIC, "non-finite Lanczos scalars");
    if (j == 0) {
        omega_[0].assign(static_cast<size_t>(m_) + 2, 0.0);
        omega_[1].assign(static_cast<size_t>(m_) + 2, 0.0);
        omega_[1][0] = 1.0;                  // row 0: <v_0, v_0>
        anorm_ = 0.0;
        force_next_ = false;
    }
    anorm_ = std::max({anorm_, std::fabs(ha_[j]), hb_[j]});
    const double bj = hb_[j];
    std::vector<double> next(static_cast<size_t>(m_) + 2, 0.0);
    double worst = 0.0;
    if (bj > 0.0) {
        const std::vector<double> &cur = omega_[1], &prev = omega_[0];
        for (int k = 0; k < j; ++k) {
            double t = hb_[k] * cur[k + 1] + (ha_[k] - ha_[j]) * cur[k];
            if (k > 0) t += hb_[k - 1] * cur[k - 1];
            if (j > 0) t -= hb_[j - 1] * prev[k];
            t += std::copysign(2.0 * eps * anorm_, t);
            next[k] = t / bj;
            worst = std::max(worst, std::fabs(next[k]));
        }
    }
    next[j] = eps;
    next[j + 1] = 1.0;
    const bool due = force_next_ || worst > std::sqrt(eps);
    force_next_ = due && !force_next_;
    if (due)
        for (int k = 0; k <= j; ++k) next[k] = eps;
    omega_[0].swap(omega_[1]);
    omega_[1].swap(next);
    return due;
}

// largest fraction f <= remaining with err(f) <= tol f (bisection in log f)
template <typename T>
template <typename E>
double KrylovRun<T>::bisect(const E &err, double remaining, double tol) {
    double lo = 0.0, hi = remaining;
    for (int it = 0; it < 200; ++it) {
        const double mid = (lo == 0.0) ? hi * 0.5 : std::sqrt(lo * hi);
        if (err(mid) <= tol * mid)
            lo = mid;
        else
            hi = mid;
        if (lo > 0.0 && hi / lo < 1.0 + 1e-3) break;
        if (lo == 0.0 && hi < 1e-14 * remaining) break;
    }
    if (lo <= 1e-12 * remaining) fail(SYK_ENOTCONV, "Krylov step size underflow (tolerance too strict)");
    return lo;
}

// whether two vectors share some of their amplitudes, but are not the same vector
template <typename T>
static bool overlap_in_part(const T *a, const T *b, uint64_t n) {
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa != pb && (pa > pb ? pa - pb : pb - pa) < n * 2 * sizeof(T);
}

// out = v; through slot 0 where they overlap in part, as the copy's threads run in no order
template <typename T>
void KrylovRun<T>::copy(const T *v, T *out) {
    if (out == v) return;
    const bool via = overlap_in_part(v, out, n_);
    if (via) launch_scale_copy<T>(v, vec(0), n_, 1.0, s_);
    launch_scale_copy<T>(via ? vec(0) : v, out, n_, 1.0, s_);
}

template <typename T>
void KrylovRun<T>::run(std::complex<double> z, const T *v, T *out, const syk_krylov_opts &o, syk_krylov_stats &st) {
    if (z == std::complex<double>(0.0, 0.0)) {
        norm(v);                                   // refuses a non-finite vector
        copy(v, out);
    } else if (o.reorth == 0 && !plain_) {
        run_fused(z, v, out, o, st);
    } else {
        run_plain(z, v, out, o, st);
    }
}

// One fused Lanczos step: the apply, whose epilogue forms y = H v_j - beta_{j-1} v_{j-1} and the partial
// sums of alpha_j, and one pass that writes u_{j+1} = y - alpha_j v_j unnormalised with the
// partial sums of its norm (the scales 1 / n_i enter wherever a slot is read).  Who adds the partials up:
//   gather kernels and, up to 2^21 amplitudes, the tiled ones: each reader (two launches a step);
//   larger: launches of their own (too many partials for every workgroup to add).
// Measured with the host following through pinned scalars instead of copies and stream waits:
// N = 26, complex128 (12 steps) 582 -> 152 us a propagation, N = 40, complex128 (27 steps) 2187 ->
// 1383 us; from N = 50 on the apply is nearly all of it (17.9 -> 17.2 ms).
template <typename T>
void KrylovRun<T>::enqueue(int j, const T *u0) {
    const T *u = j == 0 ? u0 : vec(j);
    T *w = vec(j + 1);
    LanczosFuse<T> lf;
    lf.vprev = j == 0 ? nullptr : j == 1 ? u0 : vec(j - 1);
    lf.vcur = u;
    lf.norm2 = beta2_;
    lf.j = j;
    lf.partials = fused_;
    lf.norm_parts = norms_;
    lf.n_parts = big_ ? 0 : n_norm_;
    lf.norm2_host = host_.dev(host_.norm2(j));
    pending_ = true;
    if (timer_) timer_->begin(s_);
    const int np = apply_block_lanczos<T>(h_, blk_, rot_, tiled_, u, w, lf, s_);
    if (timer_) timer_->end(s_);
    double *al = alpha_ + j, *al_host = host_.dev(host_.alpha(j));
    const bool reduce = !big_ && np <= kNormParts;
    if (!reduce) launch_publish_sum(fused_, np, al, al_host, s_);
    double *parts = big_ ? fused_ : norms_;                      // fused_ is free once alpha_j is formed
    launch_lanczos_residual<T>(w, u, al, al_host, fused_, reduce ? np : 0, beta2_, j, n_, parts, n_norm_, s_);
    if (big_) launch_publish_sum2(parts, n_norm_, partials_, beta2_ + j + 1, host_.dev(host_.norm2(j + 1)), s_);
    // otherwise the next apply sums the norm
}

// One launch per step: H u_j alternates between slot 0 and slot m, which hold no basis vector while the
// steps run, and the sums between two halves of the partials' space.
template <typename T>
LanczosStep<T> KrylovRun<T>::step_of(int j, const T *u0) {
    LanczosStep<T> st;
    T *g[2] = {basis_, vec(m_)};
    double *sums[2] = {fused_, fused_ + 3 * kStepGroups};
    st.j = j;
    st.g = j == 0 ? u0 : g[(j - 1) & 1];
    st.u1 = j == 0 ? nullptr : j == 1 ? u0 : vec(j - 1);
    st.u2 = j < 2 ? nullptr : j == 2 ? u0 : vec(j - 2);
    st.u = j == 0 ? nullptr : vec(j);
    st.gout = g[j & 1];
    st.parts = sums[(j - 1) & 1];
    st.np = n_step_;
    st.out = sums[j & 1];
    st.norm2 = beta2_;
    st.alpha = alpha_;
    if (j > 0) {
        st.norm2_host = host_.dev(host_.norm2(j - 1));
        st.alpha_host = host_.dev(host_.alpha(j - 1));
    }
    return st;
}

template <typename T>
void KrylovRun<T>::enqueue_one(int j, const T *u0) {
    pending_ = true;
    if (timer_) timer_->begin(s_);
    n_step_ = apply_step<T>(h_, blk_, step_of(j, u0), s_);
    if (timer_) timer_->end(s_);
}

// alpha_{j-1} and the norm of u_j, with no step j enqueued
template <typename T>
void KrylovRun<T>::close(int j, const T *u0) {
    LanczosStep<T> st = step_of(j, u0);
    st.next_host = host_.dev(host_.norm2(j));
    launch_lanczos_close<T>(st, static_cast<uint32_t>(n_), s_);
}

// The step after k at which the error estimate is formed: each one for large vectors, where a step
// in vain costs the most, and ever wider apart below 2^20 amplitudes.
template <typename T>
int KrylovRun<T>::next_check(int k) const {
    if (n_ >= (1ULL << 20)) return std::min(k + 1, m_);
    return std::min(k == 0 ? 4 : k + std::max(2, k / 4), m_);
}

template <typename T>
void KrylovRun<T>::run_fused(std::complex<double> z, const T *v, T *out, const syk_krylov_opts &o,
                             syk_krylov_stats &st) {
    // the two-stage sum of large blocks stages 512 doubles in partials_
    if (big_ && static_cast<size_t>(n_part_) * 2 * (m_ + 2) < 512)
        fail(SYK_EDEVICE, "partials buffer too small");
    double remaining = 1.0;
    const T *cur = v;
    // Vector 0 of the recombination is `cur` itself, read and written by the same thread where it is
    // `out`.  Where the two overlap in part a thread would write amplitudes that another has yet to
    // read: the sub-step then starts from a normalised copy in slot 0, which only one-launch
    // steps use otherwise.  So does one from a vector outside the range of the fused steps.
    bool staged = overlap_in_part(v, static_cast<const T *>(out), n_);
    std::vector<double> al(m_ + 1), n2(m_ + 2), bo(m_ + 1), coef(2 * (m_ + 1));
    std::vector<std::complex<double>> c(m_ + 1);
    while (remaining > 0.0) {
        if (o.max_substeps > 0 && st.substeps >= o.max_substeps)
            fail(SYK_ENOTCONV, "Krylov propagation exceeded max_substeps");
        const T *u0 = cur;
        double unit = 1.0;                       // cur = unit u0
        if (staged) {
            unit = norm(cur);
            if (unit == 0.0) {
                copy(cur, out);
                break;
            }
            launch_scale_copy<T>(cur, vec(0), n_, 1.0 / unit, s_);
            u0 = vec(0);
        }
        const bool one = one_ && !staged;
        host_.next();
        pending_ = true;
        if (one) {
            // step 0 sums the norm
        } else if (!big_) {
            launch_norm2_partials<T>(u0, n_, norms_, n_norm_, s_);
        } else {
            launch_norm2_partials<T>(u0, n_, partials_, n_part_, s_);
            launch_publish_sum(partials_, n_part_, beta2_, host_.dev(host_.norm2(0)), s_);
        }
        int k = 0, enq = 0;        // steps read back, enqueued
        bool again = false;
        double tau = 0.0, nrm = 0.0;
        int check = next_check(0);               // the error estimate is formed at these steps
        // log error estimates of the last three checks, newest first, and the steps between them:
        // the check at which the estimate meets the tolerance is extrapolated from them (the decay
        // steepens, so the last slope and its change are used)
        double e0 = 0.0, e1 = 0.0, e2 = 0.0;
        int d0 = 1, d1 = 1, checks = 0;
        int converges = m_;        // that check, as far as known
        for (;;) {
            // Steps are enqueued ahead of the check, so that the GPU does not wait for the host:
            // two where a step takes microseconds, one for large blocks, none beyond the check
            // expected to converge (a step enqueued in vain costs its whole time).
            // With one launch per step the norm that the check needs comes with the second step after it.
            if (one) {
                const int ahead = converges <= check || check + 2 > m_ ? check : check + 2;
                while (enq < ahead) enqueue_one(enq++, u0);
                if (enq == check) close(check, u0);
            } else {
                const int ahead = std::min(check + (big_ ? 1 : 2), std::max(check, converges));
                while (enq < std::min(ahead, m_)) enqueue(enq++, u0);
                if (!big_ && enq == check)           // no later step to sum this norm
                    launch_publish_sum(norms_, n_norm_, beta2_ + enq, host_.dev(host_.norm2(enq)), s_);
            }
            if (k == 0) {
                n2[0] = host_.wait(host_.norm2(0), s_);
                if (!std::isfinite(n2[0])) fail(SYK_ENUMERIC, "non-finite norm in Krylov propagation");
                nrm = std::sqrt(n2[0]);
                again = !staged && nrm > 0.0 && !fused_norm<T>(nrm);
                if (again) break;
            }
            const int step = check - k;
            for (; k < check; ++k) {
                al[k] = host_.wait(host_.alpha(k), s_);
                n2[k + 1] = host_.wait(host_.norm2(k + 1), s_);
            }
            if (nrm == 0.0) break;
            // beta_k ~ 0 ends the sequence at k, also between two checks
            double tnorm = 0.0, bk = 0.0;
            bool breakdown = false;
            for (int i = 0; i < k; ++i) {
                if (!std::isfinite(al[i])) fail(SYK_ENUMERIC, "non-finite Lanczos alpha");
                tnorm = std::max(tnorm, std::fabs(al[i]));
                if (i > 0) tnorm = std::max(tnorm, bo[i - 1]);
                bo[i] = bk = std::sqrt(n2[i + 1]);
                if (!std::isfinite(bk)) fail(SYK_ENUMERIC, "non-finite Lanczos beta");
                breakdown = bk <= 1e-14 * std::max(tnorm, 1e-300);
                if (breakdown) k = i + 1;
            }
            const TriLast tl(k, al.data(), bo.data());
            if (!tl.ok()) fail(SYK_ENUMERIC, "tridiagonal eigensolver failed");
            auto err = [&](double f) { return breakdown ? 0.0 : bk * tl.last(f * z); };
            const double e = err(remaining);
            if (e <= o.tol * remaining) {
                tau = remaining;
                if (breakdown) st.breakdown = 1;
                break;
            }
            if (k == m_) {
                tau = bisect(err, remaining, o.tol);
                break;
            }
            e2 = e1;
            e1 = e0;
            e0 = std::log(e);
            d1 = d0;
            d0 = step;
            check = next_check(k);
            converges = m_;
            if (++checks >= 3) {
                const double s0 = (e0 - e1) / d0, slope = std::min(s0, 2.0 * s0 - (e1 - e2) / d1);
                const double left = e0 - std::log(o.tol * remaining);
                if (slope < 0.0 && left < -slope * (m_ - k)) {
                    const int at = k + static_cast<int>(std::ceil(left / -slope));
                    for (converges = check; converges < at && converges < m_;) converges = next_check(converges);
                }
            }
        }
        if (again) {
            staged = true;
            continue;
        }
        if (nrm == 0.0) {                            // e^{zH} 0 = 0
            copy(cur, out);
            break;
        }
        st.matvecs += k;
        const TriExp te(k, al.data(), bo.data());
        if (!te.ok()) fail(SYK_ENUMERIC, "tridiagonal eigensolver failed");
        te.apply(tau * z, c.data());
        st.err_est += n2[k] <= 0.0 ? 0.0 : std::sqrt(n2[k]) * std::abs(c[k - 1]);
        for (int i = 0; i < k; ++i) {
            // slot i holds u_i = n_i v_i
            const double ni = std::sqrt(n2[i]);
            const double sc = ni > 1e-300 ? unit * nrm / ni : 0.0;
            coef[2 * i] = sc * c[i].real();
            coef[2 * i + 1] = sc * c[i].imag();
        }
        if (k <= kCombineArgs) {
            launch_combine_args<T>(u0, basis_, vec_stride_, k, coef.data(), out, n_, s_);
        } else {
            SYK_HIP(hipMemcpyAsync(coef_, coef.data(), 2 * k * sizeof(double), hipMemcpyHostToDevice, s_));
            launch_combine<T>(u0, basis_, vec_stride_, k, coef_, out, n_, s_);
        }
        st.substeps += 1;
        remaining -= tau;
        if (remaining <= 1e-15) break;
        cur = out;
        staged = false;
    }
    if (timer_) {
        SYK_HIP(hipStreamSynchronize(s_));
        timer_->flush();
    }
}

template <typename T>
void KrylovRun<T>::run_plain(std::complex<double> z, const T *v, T *out, const syk_krylov_opts &o, syk_krylov_stats &st) {
    double nrm = norm(v);
    if (nrm == 0.0) {
        copy(v, out);
        return;
    }
    double remaining = 1.0;
    const T *cur = v;
    std::vector<double> ha(2 * (m_ + 2)), hb(m_ + 2);
    std::vector<std::complex<double>> c(m_ + 1);
    std::vector<double> coef(2 * (m_ + 1));
    while (remaining > 0.0) {
        if (o.max_substeps > 0 && st.substeps >= o.max_substeps)
            fail(SYK_ENOTCONV, "Krylov propagation exceeded max_substeps");
        launch_scale_copy<T>(cur, vec(0), n_, 1.0 / nrm, s_);
        SYK_HIP(hipMemsetAsync(beta2_, 0, sizeof(double), s_));
        int k = 0;                 // Lanczos vectors built
        double tau = 0.0;
        bool done = false;
        int check = next_check(0);
        for (int j = 0; j < m_ && !done; ++j) {
            if (iterate(j, o.reorth)) st.reorths += 1;
            k = j + 1;
            st.matvecs += 1;
            if (k < check) continue;
            check = next_check(k);
            SYK_HIP(hipMemcpyAsync(ha.data(), alpha_, 2 * k * sizeof(double), hipMemcpyDeviceToHost, s_));
            SYK_HIP(hipMemcpyAsync(hb.data(), beta2_, (k + 1) * sizeof(double), hipMemcpyDeviceToHost, s_));
            SYK_HIP(hipStreamSynchronize(s_));
            if (timer_) timer_->flush();
            std::vector<double> al(k), bo(std::max(k - 1, 1));
            double tnorm = 0.0;
            for (int i = 0; i < k; ++i) {
                al[i] = ha[2 * i];
                if (!std::isfinite(al[i])) fail(SYK_ENUMERIC, "non-finite Lanczos alpha");
                tnorm = std::max(tnorm, std::fabs(al[i]));
            }
            for (int i = 0; i + 1 < k; ++i) {
                bo[i] = std::sqrt(hb[i + 1]);
                tnorm = std::max(tnorm, bo[i]);
            }
            const double bk = std::sqrt(hb[k]);
            if (!std::isfinite(bk)) fail(SYK_ENUMERIC, "non-finite Lanczos beta");
            TriExp te(k, al.data(), bo.data());
            if (!te.ok()) fail(SYK_ENUMERIC, "tridiagonal eigensolver failed");
            const bool breakdown = bk <= 1e-14 * std::max(tnorm, 1e-300);
            auto err = [&](double f) { return breakdown ? 0.0 : bk * std::abs(te.last(f * z)); };
            if (err(remaining) <= o.tol * remaining) {
                tau = remaining;
                done = true;
                if (breakdown) st.breakdown = 1;
            } else if (k == m_) {
                tau = bisect(err, remaining, o.tol);
                done = true;
            }
            if (done) {
                te.apply(tau * z, c.data());
                st.err_est += err(tau);
                for (int i = 0; i < k; ++i) {
                    coef[2 * i] = nrm * c[i].real();
                    coef[2 * i + 1] = nrm * c[i].imag();
                }
            }
        }
        // the combination writes `out`; the start vector already lives in the basis
        SYK_HIP(hipMemcpyAsync(coef_, coef.data(), 2 * k * sizeof(double), hipMemcpyHostToDevice, s_));
        launch_combine<T>(vec(0), basis_, vec_stride_, k, coef_, out, n_, s_);
        st.substeps += 1;
        remaining -= tau;
        if (remaining <= 1e-15) break;
        cur = out;
        nrm = norm(out);
        if (nrm == 0.0) break;
    }
}

template class KrylovRun<float>;
template class KrylovRun<double>;

}  // namespace syk
